"""Rows so far apart that a tile of them spans 4 GiB and more: crops of very
wide parents, and very wide images.  The stage hook and the blur sizes without
fused sweeps against one kernel per stage, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu
SIGMA = {1: 0.5, 5: 1.0, 9: 2.0, 15: 3.0}


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


def compare(hx, ks, src):
    h, w = src.shape
    with hx.Pipeline(ksize=ks, sigma=SIGMA[ks], theta=0.1, max_pixels=h * w, max_images=1,
                     forms=hx.FORM_STAGES) as p:
        for planes in (("B", "Z"), ("L", "G")):
            p.set_schedule()
            got = p.edge_detect_stages(src, stages=planes)
            p.set_schedule(64, 16, 1)
            ref = p.edge_detect_stages(src, stages=planes)
            p.sync()
            for k in ref:
                assert torch.equal(got[k], ref[k]), k
        assert bool(ref["mask"].any())
        if ks not in (3, 5, 7):
            p.set_schedule()
            assert torch.equal(p.edge_detect(src), ref["mask"])


@pytest.mark.parametrize("ks", [1, 5, 9, 15])
@pytest.mark.parametrize("pitch_log2", [25, 26, 27])
def test_crop_of_a_very_wide_parent(hx, ks, pitch_log2):
    """25: 34 rows just exceed the bound for k = 15, 26 also for the others,
    27: a few rows do."""
    h, w, pitch = 41, 203, (1 << pitch_log2) + 12
    gen = torch.Generator(device="cuda")
    gen.manual_seed(421)
    parent = torch.empty(h * pitch, device="cuda")
    src = parent.as_strided((h, w), (pitch, 1))
    src.copy_(torch.rand((h, w), generator=gen, device="cuda"))
    src[10:30, 50:150] += 2.0
    print(f"k{ks} pitch {pitch}", flush=True)
    compare(hx, ks, src)


@pytest.mark.parametrize("ks", [5, 9])
def test_very_wide_image(hx, ks):
    h, w = 20, (1 << 26) + 5
    gen = torch.Generator(device="cuda")
    gen.manual_seed(422)
    src = torch.rand((h, w), generator=gen, device="cuda")
    src[5:15, 1000:5000] += 2.0
    src[5:15, -5000:] += 2.0
    print(f"k{ks} {h}x{w}", flush=True)
    compare(hx, ks, src)

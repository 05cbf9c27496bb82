"""Images that hold both zeros, and negative values small enough to blur to
-0.0: L of a window of zeros is zero, never positive, whatever the zeros'
signs are.  Every form against one kernel per stage, bit for bit, and against
the oracle where the image's zeros are exact."""
import numpy as np
import pytest
import torch

import oracle
import parity

pytestmark = pytest.mark.gpu
THETA = 0.1
SIGMA = {1: 0.5, 3: 0.8, 5: 1.0, 7: 1.5, 9: 2.0}
H, W = 210, 707   # three 256-column tiles, one of them inside the image


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


def scenes():
    rng = np.random.default_rng(401)
    step = np.full((H, W), -0.0, np.float32)
    for x in range(20, W, 45):        # -0, a column of +0, then bright
        step[:, x] = 0.0
        step[:, x + 1:x + 9] = 1.0
        step[:, x + 9] = 0.0
    masked = rng.normal(size=(H, W)).astype(np.float32)
    masked *= (rng.random((H // 10 + 1, W // 10 + 1)) < 0.4).repeat(10, 0).repeat(10, 1)[:H, :W]
    rounded = np.round(rng.normal(scale=0.4, size=(H, W))).astype(np.float32)
    tiny = np.zeros((H, W), np.float32)
    tiny[rng.random((H, W)) < 0.2] = -1e-45
    tiny[rng.random((H, W)) < 0.05] = -3e-41
    tiny[60:90, 100:400] = 2e-20
    for im in (step, masked, rounded):
        z = im == 0
        assert (z & np.signbit(im)).any() and (z & ~np.signbit(im)).any()
    return {"step": step, "masked": masked, "rounded": rounded, "tiny": tiny}


@pytest.mark.parametrize("ks", [1, 3, 5, 7, 9])
def test_forms_agree_on_signed_zeros(hx, ks):
    imgs = scenes()
    srcs = {k: torch.from_numpy(v).cuda() for k, v in imgs.items()}
    fused = ks in (3, 5, 7)
    with hx.Pipeline(ksize=ks, sigma=SIGMA[ks], theta=THETA, max_pixels=4 * H * W) as p:
        p.set_schedule(64, 16, 1)
        ref = {k: p.edge_detect_stages(s) for k, s in srcs.items()}
        p.sync()
        forms = {"auto": None}
        if fused:
            forms.update({"short1": (64, 8, 4, hx.PASS_STORE), "short4": (256, 16, 4, hx.PASS_STORE),
                          "long": (256, 64, 4, hx.PASS_STORE), "long2": (128, 32, 4, hx.PASS_STORE),
                          "recompute": (256, 64, 4, hx.PASS_RECOMPUTE),
                          "spec16": (256, 16, 4, hx.PASS_SPECULATE),
                          "spec48": (256, 48, 4, hx.PASS_SPECULATE),
                          "depth2": (256, 32, 2, hx.PASS_STORE), "depth3": (64, 32, 3, hx.PASS_STORE)})
        for form, sched in forms.items():
            print(f"k{ks} {form}", flush=True)
            p.set_schedule(*sched) if sched else p.set_schedule()
            one = {k: p.edge_detect(s) for k, s in srcs.items()}
            many = p.edge_detect_batched(list(srcs.values()))
            for k, m in zip(srcs, many):
                assert torch.equal(one[k], ref[k]["mask"]), (form, k)
                assert torch.equal(m, ref[k]["mask"]), (form, k, "batched")
        p.set_schedule()
        for k, s in srcs.items():
            got = p.edge_detect_stages(s)
            for plane in ("B", "L", "Z", "G", "mask"):
                assert torch.equal(got[plane], ref[k][plane]), (k, plane)
    o = oracle.edge_detect(imgs["step"], ks, SIGMA[ks], THETA, stages=True)
    r = parity.compare_mask(ref["step"]["mask"].cpu().numpy(), o, THETA)
    assert o["mask"].any() and r["mismatch"] == 0, r

"""Tile sizes fixed at creation are used, also for the blur sizes whose
automatic form is another: told by the kernels a captured call holds."""
import ctypes

import pytest
import torch

from paper_2503_10855_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


def nodes(p, src, mask):
    """Graph nodes of one recorded per-image call."""
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        p.edge_detect(src, mask)
    n = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("ks", [1, 9, 13])
def test_fixed_tiles_run_the_stage_kernels(hx, ks):
    src = torch.from_numpy(synth.image(333, 450, 431, ks)).cuda()
    masks = [torch.zeros(src.shape, dtype=torch.uint8, device="cuda") for _ in range(4)]
    kw = dict(ksize=ks, sigma=0.3 * ks, theta=0.1, max_pixels=1 << 18, max_images=1)
    with hx.Pipeline(**kw) as p:
        auto = nodes(p, src, masks[0])
        p.edge_detect(src, masks[0])
        p.set_schedule(32, 16, 1)
        forced = nodes(p, src, masks[1])
        p.edge_detect(src, masks[1])
        p.sync()
    assert auto < forced
    for i, knobs in enumerate((dict(tile_w=32), dict(tile_h=32))):
        with hx.Pipeline(**kw, **knobs) as p:
            print(f"k{ks} {knobs} {p.schedule(333, 450)}", flush=True)
            assert nodes(p, src, masks[2 + i]) == forced
            p.edge_detect(src, masks[2 + i])
            p.sync()
    assert bool(masks[0].any()) and all(torch.equal(m, masks[0]) for m in masks)

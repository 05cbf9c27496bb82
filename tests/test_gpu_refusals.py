"""Calls that the interface refuses: the status, and nothing enqueued."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


@pytest.mark.parametrize("pass_mode", [-1, 4, 5])
def test_unknown_pass_structures_are_refused(hx, pass_mode):
    """A fixed depth below 4 does not look at the pass structure; the batched
    call does, and refuses a value that is none of the interface's."""
    src = torch.zeros((64, 64), device="cuda")
    mask = torch.full((64, 64), 7, dtype=torch.uint8, device="cuda")
    with hx.Pipeline(fusion_depth=2, pass_mode=pass_mode, max_pixels=1 << 14, max_images=4) as p:
        with pytest.raises(hx.HxError) as e:
            p.edge_detect_batched([src], [mask])
        assert e.value.status == hx.HX_E_INVALID
        p.sync()
        assert bool((mask == 7).all())
    with pytest.raises(hx.HxError):
        hx.Pipeline(pass_mode=pass_mode, max_pixels=1 << 14, max_images=4)

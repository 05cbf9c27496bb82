"""SRAD's short tiles (61 columns by 4, 8 or 16 rows) and upward bands where
they can go wrong: one column or row below, at and past a tile's and a
strip's edge, and sizes either side of each change of cut.  Tolerances: those
of the other SRAD tests (3e-6 max|J| per iteration against the fp64 oracle,
q0^2 within 1e-5, the two forms equal bit for bit)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_10855_amd import synth

pytestmark = pytest.mark.gpu
LAM = 0.5
SHAPES = [(3, 31), (3, 32), (4, 60), (5, 61), (8, 62), (9, 122), (1, 123), (16, 183),
          (128, 1024), (129, 1024), (1024, 1536), (1537, 1024), (1536, 2048), (1793, 1801),
          (3000, 1100)]


@pytest.mark.parametrize("shape", SHAPES)
def test_srad_cut_edges(shape):
    from paper_2503_10855_amd import hx
    img = synth.speckle(*shape, index=shape[0] + shape[1])
    niter = 3
    ref, qref = oracle.srad(img, niter, LAM)
    out = {}
    with hx.Pipeline(max_pixels=img.size, max_images=1,
                     forms=hx.FORM_STAGES | hx.FORM_SRAD) as p:
        for fused in (True, False):
            for pad in (0, 3):
                buf = torch.zeros((shape[0], shape[1] + pad), device="cuda")
                J = buf[:, :shape[1]]
                J.copy_(torch.from_numpy(img))
                q = torch.zeros(niter, dtype=torch.float64, device="cuda")
                print(f"srad {shape} fused {fused} pad {pad}", flush=True)
                p.srad(J, niter, LAM, fused=fused, q_log=q)
                torch.cuda.synchronize()
                assert int((buf[:, shape[1]:] != 0).sum()) == 0
                out[fused, pad] = (J.cpu().numpy(), q.cpu().numpy())
    J, q = out[True, 0]
    for a, b in out.values():
        assert np.array_equal(a, J) and np.array_equal(b, q)
    scale = np.abs(ref).max()
    assert np.abs(J.astype(np.float64) - ref).max() <= 3e-6 * niter * scale
    assert np.all(np.abs(q - qref) <= 1e-5 * np.abs(qref) + 1e-12)

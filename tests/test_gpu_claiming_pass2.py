"""SPECULATE's second kernel for its last pass, which the batch tuner may
choose: loaded from a cache that names it, the masks and maxima of RECOMPUTE,
bit for bit, with complete lists and with lists that overflow."""
import json

import numpy as np
import pytest
import torch

from paper_2503_10855_amd import synth

pytestmark = pytest.mark.gpu
SIGMA = {3: 0.8, 5: 1.0, 7: 1.5}


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


@pytest.mark.parametrize("ks", [3, 5, 7])
@pytest.mark.parametrize("ty", [32, 80])
def test_claiming_pass2_matches_recompute(hx, tmp_path, ks, ty):
    hidden = synth.image(1000, 1030, 461, ks, n_rect=0)
    hidden[40:60, 500:530] = 9.0     # between the sampled bands: every list overflows
    imgs = [hidden, synth.image(333, 251, 461, 1), synth.image(1, 70, 461, 2)]
    srcs = [torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda() for x in imgs]
    px, n = sum(x.size for x in imgs), len(imgs)
    cache = tmp_path / "tune.jsonl"
    cache.write_text(json.dumps({"batch": {
        "ksize": ks, "px_log2": px.bit_length() - 1, "n_log2": n.bit_length() - 1,
        "tile_h": ty, "pass": 3, "claim": 1, "tput_ms": 0.1}}) + "\n")
    with hx.Pipeline(ksize=ks, sigma=SIGMA[ks], theta=0.1, max_pixels=px, max_images=n) as p:
        p.set_schedule(256, 64, 4, hx.PASS_RECOMPUTE)
        want_m = torch.zeros(n, device="cuda")
        want = p.edge_detect_batched(srcs, dmax=want_m)
        p.set_schedule()
        p.autotune_load(str(cache))
        for call in range(3):
            print(f"k{ks} {ty} rows call {call}", flush=True)
            dm = torch.zeros(n, device="cuda")
            got = p.edge_detect_batched(srcs, dmax=dm)
            p.sync()
            assert torch.equal(dm, want_m)
            assert all(torch.equal(a, b) for a, b in zip(got, want))

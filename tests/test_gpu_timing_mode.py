"""Timing mode times the kernels that an ordinary batched call launches, and
batched calls only."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2503_10855_amd import synth

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A small and a larger batch, untimed and timed.
CHILD = """
import sys, torch
sys.path.insert(0, sys.argv[1])
from paper_2503_10855_amd import hx, synth
with hx.Pipeline(theta=0.1, max_pixels=1 << 24, max_images=8) as p:
    for shapes in ([(64, 100), (200, 150)], [(1080, 1920)] * 4):
        srcs = [torch.from_numpy(synth.image(h, w, 451, i)).cuda()
                for i, (h, w) in enumerate(shapes)]
        out = []
        for timed in (False, True):
            p.set_timing(timed)
            for _ in range(3):
                dm = torch.zeros(len(srcs), device="cuda")
                out.append((p.edge_detect_batched(srcs, dmax=dm), dm))
            if timed:
                ms = p.last_timing()
                assert all(0 <= t < 100 for t in ms) and ms[1] > 0 and ms[2] > 0, ms
        p.sync()
        for masks, dm in out[1:]:
            assert torch.equal(dm, out[0][1])
            assert all(torch.equal(a, b) for a, b in zip(masks, out[0][0]))
"""


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


def test_timed_batches_take_the_form_of_untimed_ones():
    env = dict(os.environ, HX_LOG="1")
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT], env=env, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-3000:]
    calls = [line.split(",")[2].strip() for line in r.stderr.splitlines()
             if line.startswith("[hx] batched call")]
    assert calls == ["short"] * 6 + ["SPECULATE"] * 6, calls


def test_per_image_calls_are_not_batched_calls(hx):
    """A large image takes the batch kernels by its size alone; the last
    timing stays that of the last batched call."""
    big = torch.from_numpy(synth.image(3200, 4001, 452, 0, n_rect=16)).cuda()
    small = torch.from_numpy(synth.image(300, 200, 452, 1)).cuda()
    with hx.Pipeline(theta=0.1, max_pixels=big.numel(), max_images=2) as p:
        assert p.schedule(*big.shape)[3] == hx.PASS_SPECULATE
        p.set_timing(True)
        p.edge_detect(big)
        with pytest.raises(hx.HxError):
            p.last_timing()
        p.edge_detect_batched([small])
        ms = p.last_timing()
        for _ in range(5):
            p.edge_detect(big)
        assert p.last_timing() == ms

"""Timing mode times the kernels that an ordinary batched call launches."""
import os
import subprocess
import sys

import pytest

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


def test_timed_batches_take_the_form_of_untimed_ones():
    env = dict(os.environ, HX_LOG="1")
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT], env=env, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-3000:]
    calls = [line.split(",")[2].strip() for line in r.stderr.splitlines()
             if line.startswith("[hx] batched call")]
    assert calls == ["short"] * 6 + ["SPECULATE"] * 6, calls

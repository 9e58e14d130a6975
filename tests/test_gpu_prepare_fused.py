"""The device factorisation with a block of Lanczos iterations per launch
against one kernel per step: the same factors bit for bit, at Gram sizes
around the rows per workgroup, the group width and the largest that fits, with
more rows than columns and with one group."""

import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import say

pytestmark = pytest.mark.gpu


# (D, H, G, rank, nz ratio); the Gram size is min(4 H / G, D + H)
@pytest.mark.parametrize("D,H,G,rank,p", [
    (5, 1, 4, 2, 0.0), (9, 7, 4, 9, 0.5), (40, 8, 4, 10, 0.5), (64, 31, 4, 6, 0.75), (64, 33, 4, 40, 0.5),
    (300, 129, 4, 5, 0.9), (200, 255, 4, 4, 0.5), (513, 257, 4, 4, 0.75), (100, 500, 4, 3, 0.5),
    (700, 512, 4, 35, 0.75), (60, 128, 1, 4, 0.5), (90, 120, 1, 5, 0.5), (30, 514, 4, 2, 0.5),
])
def test_fused_blocks_equal_stepwise(D, H, G, rank, p):
    w = synth.make(D, H, 1, 1, index=101)
    say("factorise D", D, "H", H, "G", G, "rank", rank)
    ms = [B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=p, groups=G,
                                flags=B.FLAG_DEVICE_FACTORISE | B.FLAG_KEEP_UNPRUNED | f) for f in (0, B.FLAG_STEPWISE)]
    assert ms[0].info["eff_rank"] == ms[1].info["eff_rank"]
    same_factors(ms, G)


# one group's factorisation, and one with many workgroups and terms
@pytest.mark.parametrize("D,H,G,rank,p", [(60, 128, 1, 4, 0.5), (700, 512, 4, 9, 0.75), (64, 33, 4, 40, 0.5)])
def test_a_wait_given_up_changes_no_factor(D, H, G, rank, p):
    """The waits of the block launches end at the first look: whatever a workgroup makes of it, the
    factors are those of the stepwise kernels, to which the host returns."""
    w = synth.make(D, H, 1, 1, index=102)
    say("given-up waits D", D, "H", H, "G", G, "rank", rank)
    ms = [B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=p, groups=G,
                                flags=B.FLAG_DEVICE_FACTORISE | B.FLAG_KEEP_UNPRUNED | f)
          for f in (B.FLAG_GIVE_UP, B.FLAG_STEPWISE)]
    same_factors(ms, G)


def test_the_thread_budget_holds_for_the_eigenpairs():
    """With OMP_NUM_THREADS=1 a device factorisation of four groups starts no threads for them."""
    code = """
import os, numpy as np
from paper_1905_00689_amd import binding as B
W = np.random.default_rng(1).normal(size=(128, 96)).astype(np.float32)
def threads(groups):
    B.approx_lstm_prepare(W[:, :64], W[:, 64:], None, 64, 32, 3, prune_ratio=0.5, groups=groups,
                          flags=B.FLAG_DEVICE_FACTORISE)
    return len(os.listdir("/proc/self/task"))
threads(1)   # one group: the runtime's own threads
print("threads", threads(1), threads(4), threads(4))
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], cwd=root, env=dict(os.environ, OMP_NUM_THREADS="1"),
                         capture_output=True, text=True, timeout=100)
    say(out.stdout, out.stderr[-500:])
    n = out.stdout.split("threads ")[1].split()
    assert n[0] == n[1] == n[2], n


def same_factors(ms, G):
    for g in range(G):
        for get in (B.approx_lstm_get_factors, B.approx_lstm_get_factors_f64):
            a, b = (get(m, g) for m in ms)
            for k in a:
                assert np.array_equal(a[k], b[k]), (g, k)

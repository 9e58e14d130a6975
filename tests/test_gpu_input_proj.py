"""The input projection's tiles: which one runs depends on the number of terms
and of (t, b) pairs, the order of its sums does not, so a sequence's output is
the same alone and beside others, bit for bit; and it matches the oracle."""

import numpy as np
import pytest
import torch

import oracle
from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import exported_factors, rel_err, run_gpu, say

pytestmark = pytest.mark.gpu
TOL = 1e-4


# (D, rank): 16-byte rows or not, x too wide for 8 pairs (D > 5120) and for 4
# (D > 10240); batches from one pair per chunk to several chunks per workgroup
@pytest.mark.parametrize("D,rank,T,Bs", [
    (260, 190, 17, (1, 3, 8, 40)),
    (259, 33, 9, (1, 8, 64)),
    (5200, 40, 5, (1, 7, 30)),
    (10300, 8, 4, (1, 5)),
])
def test_tiles_share_one_order(D, rank, T, Bs):
    H = 48
    w = synth.make(D, H, T, max(Bs), index=97)
    say("input projection D", D, "rank", rank)
    m = B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=0.5,
                              flags=B.FLAG_DEVICE_FACTORISE)
    f = exported_factors(m)
    first = None
    for Bn in Bs:
        x = np.ascontiguousarray(w.x[:, :Bn])
        h, _ = run_gpu(m, x, [rank])
        ho, _ = oracle.run(f, w.b, x, [rank])
        assert rel_err(h, ho) < TOL, Bn
        first = h[:, :, 0] if first is None else first
        assert np.array_equal(h[:, :, 0], first), Bn

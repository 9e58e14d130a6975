"""The pair kernel where the slots or units do not divide by the group's width,
at one and two timesteps (a run that is over after one exchange) and on the
same model again and again: every run equals the general kernel bit for bit."""

import numpy as np
import pytest

from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import run_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,Bn,rank,p,levels,blocks", [
    (64, 32, 1, 96, 0.5, [1, 4, 16, 96], 0),
    (50, 100, 9, 20, 0.5, [20], 0),
    (300, 203, 1, 64, 0.5, [64], 0),
    (100, 203, 1, 40, 0.5, [40], 77),      # over several XCDs
    (64, 2000, 1, 300, 0.9, [300], 0),     # over the device
    (64, 512, 1, 510, 0.5, [510], 0),      # over several XCDs because it is short
])
def test_uneven_shares_equal_general_kernel(D, H, Bn, rank, p, levels, blocks):
    w = synth.make(D, H, 2, Bn, index=73)
    say("uneven shares D", D, "H", H, "B", Bn, "levels", levels, "blocks", blocks)
    m = B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=p, flags=B.FLAG_DEVICE_FACTORISE)
    rng = np.random.default_rng(8)
    h0 = rng.normal(size=(Bn, H)).astype(np.float32) * 0.3
    c0 = rng.normal(size=(Bn, H)).astype(np.float32)
    for T in (1, 2):
        x = np.ascontiguousarray(w.x[:T])
        B.approx_lstm_set_launch(m, 0)
        B.approx_lstm_set_recurrence(m, 1)
        ref = run_gpu(m, x, levels, h0, c0, want_c=True)
        B.approx_lstm_set_recurrence(m, 0)
        B.approx_lstm_set_launch(m, blocks)
        assert B.approx_lstm_plan(m, T, Bn, levels)["pair_kernel"] == 1
        for _ in range(6):
            h, c = run_gpu(m, x, levels, h0, c0, want_c=True)
            assert np.array_equal(h, ref[0]) and np.array_equal(c, ref[1])

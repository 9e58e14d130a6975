"""The static scratch of approx_lstm_run_noalloc is shared by runs of every
layout: floats that one of them leaves (projections, exchange slots) must never
count as tagged words or flags of another, whatever launch sequence number the
other has; nor those of a captured run's last replay."""

import numpy as np
import pytest
import torch

from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import prep, say

pytestmark = pytest.mark.gpu


def general_bulk(index):
    """A run of the general kernel with the bulk exchange of h (8 x 300 values a timestep)."""
    w = synth.make(16, 300, 3, 8, index=index)
    m = prep(w, 4, 0.5)
    B.approx_lstm_set_recurrence(m, 1)
    assert B.approx_lstm_plan(m, 3, 8, [4])["bulk_h"] == 1
    return w, m


def test_floats_of_other_runs_at_every_sequence_number():
    w, m = general_bulk(76)
    wp = synth.make(16, 64, 40, 8, index=77)
    mp = prep(wp, 16, 0.5)
    assert B.approx_lstm_plan(mp, 40, 8, [16])["pair_kernel"] == 1
    x, xp = torch.from_numpy(w.x).cuda(), torch.from_numpy(wp.x).cuda()
    h, hp = torch.empty(1, 3, 8, 300, device="cuda"), torch.empty(1, 40, 8, 64, device="cuda")
    B.approx_lstm_run(m, x, [4], h)
    ref, bad, n = h.clone(), torch.zeros((), dtype=torch.int64, device="cuda"), 0
    # the sequence number is the call's, mod 65535; floats of magnitude 2^-7 to 2 have upper halves 0x3C00 to
    # 0x3FFF and 0xBC00 to 0xBFFF, an empty slot 0xFFFF (calls from other tests shift both by their number)
    near = lambda s: any(lo - 300 <= s <= hi + 300 for lo, hi in ((0x3C00, 0x3FFF), (0xBC00, 0xBFFF), (0xFFFF, 0xFFFF)))
    for seq in range(0x10000 + 600):
        if seq % 8192 == 0:
            say("call", seq)
        if near(seq) and seq & 1:
            h.zero_()
            B.approx_lstm_run_noalloc(m, x, [4], h)
            bad += (h != ref).any()
            n += 1
        else:
            B.approx_lstm_run_noalloc(mp, xp, [16], hp)
    B.approx_lstm_check(m)
    B.approx_lstm_check(mp)
    assert n > 1500 and int(bad) == 0, int(bad)


def test_replays_of_the_general_kernel():
    w, m = general_bulk(78)
    xs = [torch.from_numpy(np.ascontiguousarray(np.roll(w.x, i, axis=2))).cuda() for i in range(3)]
    x, h, want = xs[0].clone(), torch.empty(1, 3, 8, 300, device="cuda"), []
    for v in xs:
        B.approx_lstm_run_noalloc(m, v, [4], h)
        want.append(h.clone())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.approx_lstm_run_noalloc(m, x, [4], h)
    for i in (0, 1, 2, 1, 1, 0):
        x.copy_(xs[i])
        h.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(h, want[i]), i
        other = torch.empty_like(h)
        B.approx_lstm_run_noalloc(m, xs[2], [4], other)
        assert torch.equal(other, want[2])
    B.approx_lstm_check(m)

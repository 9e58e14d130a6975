"""The start of a group of workgroups: its words carry the launch's tag, and the
kernel before it on its stream clears them, so that a captured launch may be
replayed with the tag it was captured with, and a run of one timestep (over after
one exchange, in which some workgroups may have no part) leaves nothing behind
that the next run could mistake for its own."""

import numpy as np
import pytest
import torch

from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import prep, say

pytestmark = pytest.mark.gpu


def calls(D, H, T, Bn, rank, p):
    """(name, run(x, h)) of the register kernels: pair, exact and batched."""
    w = synth.make(D, H, T, Bn, index=75)
    m, b = prep(w, rank, p), prep(w, rank, p, factor_dtype=1)
    e = B.approx_lstm_exact_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H)
    assert B.approx_lstm_plan(m, T, Bn, [rank])["pair_kernel"] == 1
    return w, [("pair", lambda x, h: B.approx_lstm_run_noalloc(m, x, [rank], h[None]), lambda: B.approx_lstm_check(m)),
               ("exact", lambda x, h: B.approx_lstm_exact_run(e, x, h), lambda: B.approx_lstm_exact_check(e)),
               ("batched", lambda x, h: B.approx_lstm_run(b, x, [rank], h[None]), lambda: B.approx_lstm_check(b))]


@pytest.mark.parametrize("D,H,T,Bn,rank,p", [(64, 100, 5, 9, 20, 0.5), (96, 512, 1, 1, 20, 0.5)])
def test_replays_equal_eager_runs(D, H, T, Bn, rank, p):
    w, runs = calls(D, H, T, Bn, rank, p)
    xs = [torch.from_numpy(np.ascontiguousarray(np.roll(w.x, i, axis=2))).cuda() for i in range(3)]
    for name, run, check in runs:
        say("replays of", name, "H", H, "T", T)
        x, h = xs[0].clone(), torch.empty(T, Bn, H, device="cuda")
        want = []
        for v in xs:
            run(v, h)
            want.append(h.clone())
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            run(x, h)
        for i in (0, 1, 2, 1, 1, 0):
            x.copy_(xs[i])
            h.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(h, want[i]), (name, i)
            other = torch.empty_like(h)
            run(xs[2], other)               # an eager run between
            assert torch.equal(other, want[2]), (name, i)
        check()


@pytest.mark.parametrize("H,T,blocks", [(512, 2, 0), (512, 2, 64), (700, 3, 0), (203, 6, 128), (203, 1, 7)])
def test_replays_of_the_exact_kernel_on_any_width(H, T, blocks):
    """exact_lstm_kernel's tagged words: two halves by parity, cleared by the projection before it; more
    workgroups than units to deal out."""
    w = synth.make(40, H, T, 2, index=79)
    m = B.approx_lstm_exact_prepare(w.W[:, :40], w.W[:, 40:], w.b, 40, H)
    B.approx_lstm_exact_set_launch(m, blocks)
    xs = [torch.from_numpy(np.ascontiguousarray(np.roll(w.x, i, axis=2)[:, :1])).cuda() for i in range(3)]
    say("exact replays H", H, "T", T, "blocks", blocks)
    x, h, want = xs[0].clone(), torch.empty(T, 1, H, device="cuda"), []
    for v in xs:
        B.approx_lstm_exact_run(m, v, h)
        want.append(h.clone())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.approx_lstm_exact_run(m, x, h)
    for i in (0, 1, 2, 1, 1, 0):
        x.copy_(xs[i])
        h.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(h, want[i]), i
        other = torch.empty_like(h)
        B.approx_lstm_exact_run(m, xs[2], other)
        assert torch.equal(other, want[2])
    B.approx_lstm_exact_check(m)


def test_one_timestep_again_and_again():
    w, runs = calls(40, 512, 1, 20, 20, 0.5)
    x = torch.from_numpy(w.x).cuda()
    for name, run, check in runs:
        say("one timestep", name)
        hs = [torch.full((1, 20, 512), float("nan"), device="cuda") for _ in range(50)]
        for h in hs:
            run(x, h)
        check()
        for h in hs[1:]:
            assert torch.equal(h, hs[0])
        assert torch.isfinite(hs[0]).all()

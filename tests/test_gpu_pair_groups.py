"""The pair kernel on groups of workgroups: several (level, sequence) pairs
side by side, more pairs than there are groups, a group that finds itself one
workgroup short at its start (one of them computes the pairs alone), a group
spread over the device, and runs on two streams at once.  Every sum has one
order, so each run equals the general kernel's bit for bit (that kernel is
checked against the oracle elsewhere)."""

import numpy as np
import pytest
import torch

from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import run_gpu, say

pytestmark = pytest.mark.gpu


def model(D, H, T, Bn, rank, p, groups=4, index=71):
    w = synth.make(D, H, T, Bn, index=index)
    say(f"prepare D={D} H={H} T={T} B={Bn} rank={rank} p={p} groups={groups}")
    return w, B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=p, groups=groups,
                                    flags=B.FLAG_DEVICE_FACTORISE)


def general(m, *args):
    B.approx_lstm_set_recurrence(m, 1)
    try:
        return run_gpu(m, *args, want_c=True)
    finally:
        B.approx_lstm_set_recurrence(m, 0)


def same(a, b):
    return np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


# H not a multiple of 4, 16 or the group width; K = 0 beside positive budgets;
# budgets at the edges of the lane-count rule; 11 and 18 pairs (two and three
# rounds of groups); dense v; one group of terms for all gates
@pytest.mark.parametrize("D,H,T,Bn,rank,p,groups,levels", [
    (64, 32, 8, 1, 96, 0.5, 4, [1, 4, 16, 96]),
    (300, 203, 7, 3, 70, 0.5, 4, [16, 64, 7]),
    (128, 101, 6, 11, 40, 0.0, 4, [40]),
    (96, 61, 5, 9, 33, 0.75, 1, [33, 0]),
    (512, 512, 1, 8, 257, 0.9, 4, [257]),
    (200, 1024, 5, 2, 65, 0.75, 4, [63, 0, 65]),
    (256, 2048, 4, 3, 32, 0.9, 4, [32]),
])
def test_groups_equal_general_kernel(D, H, T, Bn, rank, p, groups, levels):
    w, m = model(D, H, T, Bn, rank, p, groups)
    rng = np.random.default_rng(5)
    h0 = rng.normal(size=(Bn, H)).astype(np.float32) * 0.3
    c0 = rng.normal(size=(Bn, H)).astype(np.float32)
    plan = B.approx_lstm_plan(m, T, Bn, levels)
    say("  plan", plan)
    assert plan["pair_kernel"] == 1
    ref = general(m, w.x, levels, h0, c0)
    assert same(run_gpu(m, w.x, levels, h0, c0, want_c=True), ref)
    # nobody waits: one workgroup of a group takes the pairs alone, with the same
    # bits; the next run is as before
    B.approx_lstm_set_start_wait(m, 0.0)
    assert same(run_gpu(m, w.x, levels, h0, c0, want_c=True), ref)
    B.approx_lstm_set_start_wait(m, 2000.0)
    assert same(run_gpu(m, w.x, levels, h0, c0, want_c=True), ref)


def test_group_over_the_device():
    """128 workgroups: not one XCD's, so agent-scope stores between XCDs."""
    w, m = model(256, 512, 6, 1, 300, 0.75)
    ref = general(m, w.x, [300])
    B.approx_lstm_set_launch(m, 128)
    assert B.approx_lstm_plan(m, 6, 1, [300])["blocks"] == 128
    for wait in (2000.0, 0.0, 2000.0):
        B.approx_lstm_set_start_wait(m, wait)
        assert same(run_gpu(m, w.x, [300], want_c=True), ref)


def test_runs_on_two_streams_at_once():
    """Two models, each on its own stream, many runs in flight (eight pairs
    fill the device, one pair shares it): every result is the lone run's."""
    parts = []
    for i, (Bn, K) in enumerate(((8, 64), (1, 128))):
        w, m = model(512, 512, 12, Bn, K, 0.75, index=80 + i)
        ref, _ = run_gpu(m, w.x, [K])
        x = torch.from_numpy(w.x).cuda()
        outs = [torch.full((1, 12, Bn, 512), float("nan"), device="cuda") for _ in range(20)]
        parts.append((m, x, K, ref, outs, torch.cuda.Stream()))
    torch.cuda.synchronize()
    say("two streams, 20 runs each")
    for i in range(20):
        for m, x, K, _, outs, s in parts:
            B.approx_lstm_run(m, x, [K], outs[i], stream=s)
    torch.cuda.synchronize()
    for m, _, _, ref, outs, s in parts:
        B.approx_lstm_check(m, stream=s)
        for h in outs:
            assert np.array_equal(h.cpu().numpy(), ref)


def test_stamps_of_a_lone_workgroup():
    """A timed run whose group falls back to one workgroup has that workgroup's stamps, not an earlier run's."""
    w, m = model(128, 512, 8, 1, 64, 0.75)
    B.approx_lstm_set_timing(m, 1)
    run_gpu(m, w.x, [64])
    group = B.approx_lstm_get_timing(m, 8)
    B.approx_lstm_set_start_wait(m, 0.0)
    run_gpu(m, w.x, [64])
    alone = B.approx_lstm_get_timing(m, 8)
    say("group", group[-1], "alone", alone[-1])
    assert alone[0] == 0.0 and (np.diff(alone) >= 0.0).all(), alone
    assert alone[-1] > 3.0 * group[-1]


def test_start_wait_range():
    _, m = model(64, 32, 2, 1, 4, 0.5)
    for bad in (-1.0, float("nan"), 2e7):
        with pytest.raises(B.ApproxLstmError) as ei:
            B.approx_lstm_set_start_wait(m, bad)
        assert ei.value.status == B.ERR_INVALID_ARG


# register buckets of narrow groups with much per workgroup: 17 to 32 U entries
# in each of four rows per thread (one and two phase-A passes), two passes of 24
# h-part entries; a group over several XCDs at its edges (two phase-A passes do
# not fit, a last workgroup without terms, with few units); no terms at all
# (one and several workgroups per pair, more pairs than compute units hold)
@pytest.mark.parametrize("D,H,T,Bn,rank,p,levels,blocks", [
    (64, 2048, 4, 2, 131, 0.9, [131], 0),
    (64, 1024, 5, 1, 300, 0.8, [300], 0),
    (64, 1024, 3, 3, 300, 0.95, [300, 5], 0),
    (64, 512, 5, 1, 270, 0.45, [270], 0),
    (64, 512, 6, 1, 270, 0.0, [270], 0),
    (64, 512, 3, 1, 270, 0.75, [270], 96),
    (100, 203, 5, 1, 40, 0.5, [40], 77),
    (40, 512, 5, 1, 8, 0.5, [0], 0),
    (40, 700, 3, 5, 8, 0.5, [0, 0], 0),
    (40, 96, 2, 30, 8, 0.5, [0] * 9, 0),
])
def test_wide_buckets_spread_groups_and_no_terms(D, H, T, Bn, rank, p, levels, blocks):
    w, m = model(D, H, T, Bn, rank, p)
    rng = np.random.default_rng(6)
    h0 = rng.normal(size=(Bn, H)).astype(np.float32) * 0.3
    c0 = rng.normal(size=(Bn, H)).astype(np.float32)
    ref = general(m, w.x, levels, h0, c0)
    B.approx_lstm_set_launch(m, blocks)
    plan = B.approx_lstm_plan(m, T, Bn, levels)
    say("  plan", plan)
    assert plan["pair_kernel"] == 1
    for _ in range(2):
        assert same(run_gpu(m, w.x, levels, h0, c0, want_c=True), ref)


def test_limits_do_not_depend_on_the_kernel():
    """Many pairs that the general kernel's LDS cannot hold are refused on either kernel."""
    w, m = model(40, 512, 2, 300, 8, 0.5)
    for levels in ([0], [8]):
        for kernel in (0, 1):
            B.approx_lstm_set_recurrence(m, kernel)
            with pytest.raises(B.ApproxLstmError):
                run_gpu(m, w.x, levels)

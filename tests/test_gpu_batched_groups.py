"""The persistent batched recurrence at the edges of its register buckets (4, 8
and 16 contraction steps of 32 over the units and over the terms), of its
groups (one workgroup, several groups per XCD, more cohorts than groups) and
with one group of terms for all gates; against the oracle with bf16 operands,
and every sequence's output beside different numbers of others bit for bit."""

import numpy as np
import pytest

import oracle
from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import exported_factors, rel_err, run_gpu, say

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("H,rank,G,T,Bs", [
    (32, 20, 4, 3, (16, 300)),       # one workgroup per cohort
    (129, 129, 4, 3, (17, 90)),      # five contraction steps either way
    (257, 33, 4, 2, (5, 420)),       # nine steps over the units; more cohorts than groups fit
    (128, 128, 1, 1, (33, 70)),      # one timestep
    (512, 257, 4, 3, (16, 40)),
])
def test_buckets_and_groups(H, rank, G, T, Bs):
    D = 40
    w = synth.make(D, H, T, max(Bs), index=99)
    say("batched groups H", H, "rank", rank, "G", G)
    m = B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=0.5, groups=G, factor_dtype=1,
                              flags=B.FLAG_DEVICE_FACTORISE)
    f = exported_factors(m)
    levels = [rank, 3]
    first = None
    for Bn in Bs:
        x = np.ascontiguousarray(w.x[:, :Bn])
        h, c = run_gpu(m, x, levels, want_c=True)
        n = min(Bn, 24)
        ho, co = oracle.run(f, w.b, np.ascontiguousarray(x[:, :n]), levels, operand_round="bf16")
        for j in range(len(levels)):
            assert rel_err(h[j:j + 1, :, :n], ho[j:j + 1]) < TOL, (Bn, levels[j])
            assert np.abs(c[j, :n] - co[j]).max() < TOL * max(1.0, np.abs(co[j]).max())
        again, _ = run_gpu(m, x, levels)
        assert np.array_equal(h, again)
        # beside more others (and so in other tiles of the projection, which D = 64 after padding never
        # splits, and maybe after another cohort) the sequences' bits are the same
        if first is None:
            first = h
        else:
            assert np.array_equal(h[:, :, :first.shape[2]], first)
        # the last sequence too: a cohort that ran after another on its group
        hl, _ = oracle.run(f, w.b, np.ascontiguousarray(x[:, -1:]), levels, operand_round="bf16")
        assert rel_err(h[:, :, -1:], hl) < TOL


# few terms beside many units: the first workgroup (one of 16, one of 10) owns every z tile, the others only poll
@pytest.mark.parametrize("H,rank,G,T,Bn", [(512, 20, 4, 12, 40), (300, 20, 1, 12, 330), (512, 100, 4, 2, 16)])
def test_workgroups_without_terms(H, rank, G, T, Bn):
    D = 40
    w = synth.make(D, H, T, Bn, index=97)
    say("batched, workgroups without terms H", H, "rank", rank, "G", G)
    m = B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=0.5, groups=G, factor_dtype=1,
                              flags=B.FLAG_DEVICE_FACTORISE)
    h, c = run_gpu(m, w.x, [rank], want_c=True)
    ho, co = oracle.run(exported_factors(m), w.b, w.x, [rank], operand_round="bf16")
    assert rel_err(h, ho) < TOL
    assert np.abs(c - co).max() < TOL * max(1.0, np.abs(co).max())
    for _ in range(8):
        assert np.array_equal(run_gpu(m, w.x, [rank])[0], h)


@pytest.mark.parametrize("D,H,rank,T,Bn", [
    (40, 96, 70, 16, 700),      # 3 x 88 tiles of 128 rows: the last 256-row tile is half empty, x read by elements
    # 16 x 17 tiles, the last column tile half empty, x read by float4; D = 64 is two slices, which the small call
    # does not split either (from D = 128 on it adds two partial sums, in another order than one chain)
    (64, 512, 500, 3, 700),
])
def test_wide_projection_tiles(D, H, rank, T, Bn):
    """A call with more 128-row projection tiles than compute units takes the 256-row tiles: a sequence's
    bits are those of a call small enough for the others, and agree with the oracle."""
    w = synth.make(D, H, T, Bn, index=98)
    say("wide projection tiles H", H, "rank", rank, "D", D)
    m = B.approx_lstm_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H, rank, prune_ratio=0.5, factor_dtype=1,
                              flags=B.FLAG_DEVICE_FACTORISE)
    h, _ = run_gpu(m, w.x, [rank])
    for pick in (slice(0, 20), slice(Bn - 20, Bn)):
        x = np.ascontiguousarray(w.x[:, pick])
        few, _ = run_gpu(m, x, [rank])
        assert np.array_equal(h[:, :, pick], few)
    ho, _ = oracle.run(exported_factors(m), w.b, x, [rank], operand_round="bf16")
    assert rel_err(few, ho) < TOL

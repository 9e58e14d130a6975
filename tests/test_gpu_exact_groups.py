"""The exact LSTM with W_h in registers (one sequence per XCD, or one run over
the device) against exact_lstm_kernel at a width given by the caller: the same
bits, also where one workgroup of a group runs alone, at the edges of the
layers each takes, and against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import rel_err, say

pytestmark = pytest.mark.gpu
TOL = 1e-4


def run(m, w, h0, c0, rows):
    T, Bn, H = w.T, w.B, w.H
    h = torch.full((T, Bn, H), float("nan"), device="cuda")
    c = torch.full((Bn, H), float("nan"), device="cuda")
    B.approx_lstm_exact_run_rows(m, torch.from_numpy(w.x).cuda(), rows, h, torch.from_numpy(h0).cuda(),
                                 torch.from_numpy(c0).cuda(), c)
    B.approx_lstm_exact_check(m)
    torch.cuda.synchronize()
    return h.cpu().numpy(), c.cpu().numpy()


# (H, T, B, rows): one workgroup up to 32 units; 16-unit and group edges; more
# sequences than XCDs; one timestep; the layer sizes either side of 768 and up
# to 2048; 1, 2, 3 (padded to 4) and 8 sequences over the device
@pytest.mark.parametrize("H,T,Bn,rows", [
    (1, 3, 1, 1), (17, 4, 2, 9), (32, 5, 1, 32), (33, 4, 9, 33), (129, 1, 1, 129), (250, 4, 3, 100),
    (257, 5, 1, 257), (512, 7, 8, 512), (513, 4, 2, 0), (768, 4, 1, 768), (769, 4, 1, 500), (1024, 1, 2, 1024),
    (1025, 4, 3, 1025), (2048, 4, 8, 2048),
    # more than eight sequences over the device take turns; runs too short for the registers of one XCD
    (900, 3, 19, 900), (512, 2, 1, 512), (700, 3, 1, 700), (250, 2, 1, 250),
])
def test_register_kernels_equal_any_width(H, T, Bn, rows):
    w = synth.make(24, H, T, Bn, index=95)
    rng = np.random.default_rng(3)
    h0 = rng.normal(size=(Bn, H)).astype(np.float32) * 0.5
    c0 = rng.normal(size=(Bn, H)).astype(np.float32)
    say("exact registers H", H, "T", T, "B", Bn, "rows", rows)
    m = B.approx_lstm_exact_prepare(w.W[:, :24], w.W[:, 24:], w.b, 24, H)
    B.approx_lstm_exact_set_launch(m, 128 if H > 512 else 5)
    ref = run(m, w, h0, c0, rows)
    B.approx_lstm_exact_set_launch(m, 0)
    for wait in (2000.0, 0.0, 2000.0):
        B.approx_lstm_exact_set_start_wait(m, wait)
        got = run(m, w, h0, c0, rows)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]), wait
    he, ce = oracle.row_tile_lstm(w.W, w.b, w.x, rows, h0, c0)
    assert rel_err(ref[0], he) < TOL
    assert np.abs(ref[1] - ce).max() < TOL * max(1.0, np.abs(ce).max())


def test_many_wide_sequences_are_refused_on_either_kernel():
    w = synth.make(24, 1024, 2, 64, index=94)
    m = B.approx_lstm_exact_prepare(w.W[:, :24], w.W[:, 24:], w.b, 24, 1024)
    zero = np.zeros((64, 1024), np.float32)
    for blocks in (0, 128):
        B.approx_lstm_exact_set_launch(m, blocks)
        with pytest.raises(B.ApproxLstmError) as ei:
            run(m, w, zero, zero, 1024)
        assert ei.value.status == B.ERR_UNSUPPORTED


def test_the_wide_start_outlasts_a_neighbour():
    """Another stream's products hold the compute units for tens of milliseconds when a run over the device
    starts: it waits for them instead of falling to one workgroup, which would take over a second."""
    T, Bn, H = 16, 8, 2048
    w = synth.make(24, H, T, Bn, index=96)
    m = B.approx_lstm_exact_prepare(w.W[:, :24], w.W[:, 24:], w.b, 24, H)
    zero = np.zeros((Bn, H), np.float32)
    ref = run(m, w, zero, zero, H)
    x, h = torch.from_numpy(w.x).cuda(), torch.empty(T, Bn, H, device="cuda")
    a = torch.randn(8192, 8192, device="cuda")
    a @ a
    torch.cuda.synchronize()
    other, mine = torch.cuda.Stream(), torch.cuda.Stream()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    say("wide start beside another stream's products")
    with torch.cuda.stream(other):
        ev[0].record()
        for _ in range(4):
            a @ a
        ev[1].record()
    with torch.cuda.stream(mine):
        ev[2].record()
        B.approx_lstm_exact_run(m, x, h)
        ev[3].record()
    torch.cuda.synchronize()
    B.approx_lstm_exact_check(m)
    busy, took = ev[0].elapsed_time(ev[1]), ev[2].elapsed_time(ev[3])
    say("  products ms", busy, "run ms", took)
    assert np.array_equal(h.cpu().numpy(), ref[0])
    assert took < 400.0 + 2.0 * busy

"""The x projections of the exact LSTM at the edges of their tiles: 16-row and
64-column workgroups, 128 x 128 tiles, contraction lengths that end inside a
16-byte unit, a wave's span or a staged slice, row budgets that end inside a
tile, and x that is not 16-byte aligned."""

import numpy as np
import pytest
import torch

import oracle
from paper_1905_00689_amd import synth
from paper_1905_00689_amd import binding as B

from .gpu_helpers import rel_err, say

pytestmark = pytest.mark.gpu
TOL = 1e-4


@pytest.mark.parametrize("D,H,T,Bn,rows,offset", [
    (1, 1, 1, 1, 1, 0),
    (127, 5, 16, 1, 5, 0),          # one column block of 16, 20 rows
    (128, 17, 13, 5, 3, 0),         # 65 columns: a second column block
    (2052, 16, 17, 1, 16, 0),       # past one register pass of a wave
    (2300, 33, 3, 2, 20, 1),        # unaligned x
    (70, 1024, 65, 8, 999, 0),      # tiles, D not a multiple of 4
    (68, 1030, 65, 8, 1030, 1),     # tiles, rows past a tile, unaligned x
    (64, 1024, 64, 8, 1024, 0),     # tiles, every edge exact
])
def test_x_projection_edges(D, H, T, Bn, rows, offset):
    w = synth.make(D, H, T, Bn, index=90)
    say("exact x projection", D, H, T, Bn, rows, offset)
    m = B.approx_lstm_exact_prepare(w.W[:, :D], w.W[:, D:], w.b, D, H)
    buf = torch.zeros(w.x.size + offset, device="cuda")
    buf[offset:] = torch.from_numpy(w.x.reshape(-1))
    x = buf[offset:].view(T, Bn, D)
    h = torch.full((T, Bn, H), float("nan"), device="cuda")
    B.approx_lstm_exact_run_rows(m, x, rows, h)
    B.approx_lstm_exact_check(m)
    torch.cuda.synchronize()
    he, _ = oracle.row_tile_lstm(w.W, w.b, w.x, rows)
    e = rel_err(h.cpu().numpy(), he)
    say("  rel err", e)
    assert e < TOL

"""Every workgroup of a pair-kernel group owns exchange slots of z and hidden
units.  The exchange rests on it: a slot is emptied for the next value once
everyone has published what it computed from the present one, which says
nothing about a workgroup that publishes nothing."""

import numpy as np
import pytest

from paper_1905_00689_amd import binding as B


def model(H, rank, groups=4, D=8, nz=0):
    """Host-only model of an all-zero matrix (its chain ends at once): the plan needs sizes alone."""
    W = np.zeros((4 * H, D + H), np.float32)
    return B.approx_lstm_prepare(W[:, :D], W[:, D:], None, D, H, rank, nz=nz or D + H // 4, groups=groups,
                                 flags=B.FLAG_HOST_ONLY)


def check(m, T, Bn, levels):
    """Widths of the levels; every share positive wherever something is exchanged."""
    H, G, widths = m.info["hidden_size"], m.info["groups"], []
    for i, K in enumerate(levels):
        own = B.approx_lstm_plan_shares(m, T, Bn, levels, i, num_cu=256)
        widths.append(len(own))
        if not own:
            continue
        slots, units = (sum(o[k] for o in own) for k in (0, 1))
        assert units == H and slots >= G * K, (H, levels, own)
        if len(own) > 1 and K > 0:
            assert min(min(o) for o in own) >= 1, (H, levels, own)
            assert max(o[0] for o in own) - min(o[0] for o in own) <= 1, own
            assert max(o[1] for o in own) - min(o[1] for o in own) <= 1, own
    return widths


# odd and even layers, from one wave's units to the widest; 2000 units with 300 terms spread over the device
@pytest.mark.parametrize("H", [24, 33, 61, 100, 101, 203, 333, 512, 700, 1024])
@pytest.mark.parametrize("groups", [4, 1])
def test_every_workgroup_owns_slots_and_units(H, groups):
    m = model(H, 144, groups)
    wide = 0
    for K in list(range(1, 20)) + [31, 32, 33, 48, 63, 64, 65, 96, 100, 127, 128, 129, 144]:
        for Bn in (1, 5):
            wide += check(m, 4, Bn, [K])[0] > 1
    for levels in ([1, 4, 16, 96], [144, 0, 20]):
        wide += max(check(m, 4, 1, levels)) > 1
    assert wide


def test_widths_of_the_tiny_model_and_of_spread_groups():
    assert max(check(model(32, 96, D=64, nz=48), 8, 1, [1, 4, 16, 96])) > 1
    m = model(2000, 300, nz=200)
    assert check(m, 1, 1, [300])[0] > 64
    # a width that the caller asks for: one that would leave workgroups without a share is the general kernel's
    m = model(203, 40)   # 192 slots
    for blocks in (16, 77, 96, 192, 193):
        B.approx_lstm_set_launch(m, blocks)
        assert check(m, 5, 1, [40])[0] == (blocks if blocks <= 192 else 0), blocks

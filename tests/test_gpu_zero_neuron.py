"""A sample whose amplitude is 0 (one output neuron exactly 0): f(S') - f(s) is
undefined where S' keeps the zero and +infinity where the exchange removes it,
also where AUTO recomputes only the neurons that the exchange can change."""
import numpy as np
import pytest
import torch

from paper_2204_07816_amd import nqs

pytestmark = pytest.mark.gpu
NONFINITE = 6


def cnn1_weights(C):
    """u[0] = (sum of the 3x3 spins) - 9, the other neurons 1."""
    W, a = np.zeros((2 * C, 1, 9)), np.zeros(2 * C)
    V, v = np.zeros((C, C, 9)), np.ones(C)
    W[0, 0, :], a[1] = 1.0, -20.0
    V[0, 0, 4], v[0] = 1.0, -9.0
    return np.concatenate([x.reshape(-1) for x in (W, a, V, v)])


@pytest.mark.parametrize("at", [(1, 1), (0, 4), (5, 2)])
def test_zero_outside_the_region(at):
    L, C = 6, 16
    s = -np.ones((L, L), np.int8)
    for d in np.ndindex(3, 3):                     # up on 3x3 around `at`, and far from it
        s[(at[0] + d[0] - 1) % L, (at[1] + d[1] - 1) % L] = 1
    s[(at[0] + 3) % L, (at[1] + 3) % L] = 1
    ctx = nqs.Context.cnn1(L, 1.0, 0.5, 1, C, cnn1_weights(C))
    sp = torch.as_tensor(s[None].copy()).cuda()
    counts, offs, bonds, _, _ = ctx.connected(sp)
    n = int(offs[-1])
    b = bonds[:n].cpu().numpy()
    DX, DY = np.array([1, 0, 1, 1]), np.array([0, 1, 1, -1])
    want = np.empty(n)
    for k in range(n):
        i = b[k] >> 2
        x, y = i % L, i // L
        j = ((y + DY[b[k] & 3]) % L, (x + DX[b[k] & 3]) % L)
        t = s.copy()
        t[y, x], t[j] = t[j], t[y, x]
        nine = sum(np.roll(t.astype(int), (dy, dx), (0, 1)) for dy in (-1, 0, 1) for dx in (-1, 0, 1))
        want[k] = np.nan if np.any(nine == 9) else np.inf
    assert np.isnan(want).any() and np.isinf(want).any()
    for mode in ("full", "auto"):
        d = ctx.log_ratios(sp, mode=mode)[:n].cpu().numpy()
        assert np.array_equal(d, want, equal_nan=True), mode
        assert ctx.get_error() == NONFINITE
        assert not np.isfinite(ctx.local_energy(sp, mode=mode).cpu().numpy()).any()
        assert ctx.get_error() == NONFINITE


@pytest.mark.parametrize("tj", [False, True])
def test_zero_amplitude_without_exchanges(tj):
    """All spins up: neurons of 0, but no configuration to compare with, so the
    energy is the diagonal part (spins: 72 bonds of (J1 + J2) / 4; t-J: 0)."""
    L, C = 6, 16
    w = cnn1_weights(C)
    ctx = nqs.Context.cnn1_tj(L, 1.0, 0.4, 1, C, w) if tj else nqs.Context.cnn1(L, 1.0, 0.5, 1, C, w)
    sp = torch.ones((1, L, L), dtype=torch.int8, device="cuda")
    got = []
    for mode in ("full", "auto"):
        e = float(ctx.local_energy(sp, mode=mode)[0])
        assert e == (0.0 if tj else 27.0), mode
        got.append(ctx.get_error())
    assert got[0] == got[1]

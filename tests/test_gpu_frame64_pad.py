"""The frame form with channels filled up to 16 or 32: ln cosh networks of other
channel counts, where AUTO and the Metropolis chains take it, against the
layered full recomputation, the oracle and the oracle's chains."""
import numpy as np
import pytest
import torch

import oracle
from paper_2204_07816_amd import inputs, nqs

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("L,K,C,B", [
    (4, 2, 1, 3), (4, 3, 3, 5), (4, 2, 4, 64), (6, 2, 4, 64), (6, 4, 15, 40), (8, 3, 17, 9),
    (10, 4, 8, 30), (12, 2, 5, 20), (12, 5, 24, 3), (14, 2, 8, 12), (16, 3, 31, 2), (20, 2, 7, 6),
])
def test_ratios(dtype, L, K, C, B):
    w = inputs.stress_weights(K, C, 1.0, 61)
    sp = inputs.spins_any(L, B, 62)
    spd = torch.as_tensor(sp).cuda()
    ctx = nqs.Context(L, 1.0, 0.5, K, C, w, dtype)
    for step in range(2):
        counts, offs, *_ = ctx.connected(spd)
        n = int(offs[-1])
        full = ctx.log_ratios(spd, mode="full")[:n].cpu().numpy()
        auto = ctx.log_ratios(spd, mode="auto")[:n].cpu().numpy()
        # the same neurons; FP64 sums over the sites in another order, and each a
        # difference of two sums or a sum of differences
        f = float(ctx.log_psi(spd)[0].abs().max())
        assert np.max(np.abs(full - auto)) <= 64 * EPS * max(1.0, f)
        if dtype == "fp64" and L <= 10:
            ref = oracle.local_energy(L, 1.0, 0.5, K, C, w, sp)
            e = ctx.local_energy(spd).cpu().numpy()
            assert np.max(np.abs(e - ref)) <= 1e-10 * np.max(np.abs(ref))
        # once more with the weights changed on the device
        d = np.cos(np.arange(w.size))
        ctx.update_weights(torch.as_tensor(d).cuda(), 0.01)
        w = w + 0.01 * d
    assert ctx.get_error() == 0


@pytest.mark.parametrize("L,K,C,B,steps", [
    (4, 2, 3, 5, 7), (4, 2, 4, 2500, 3), (6, 3, 8, 3, 9), (12, 2, 24, 3, 6), (14, 2, 8, 2, 5),
])
def test_chains_equal_the_oracle(L, K, C, B, steps):
    w = inputs.stress_weights(K, C, 1.0, 63)
    sp = inputs.spins_sz0(L, B, 64)
    rb, ru = inputs.mcmc_randoms(65, 0, steps, B)
    want, acc = oracle.mcmc(L, 1.0, 0.5, K, C, w, sp, rb, ru)
    ctx = nqs.Context(L, 1.0, 0.5, K, C, w)
    spd = torch.as_tensor(sp.copy()).cuda()
    got = ctx.mcmc(spd, torch.as_tensor(rb).cuda(), torch.as_tensor(ru).cuda())
    assert np.array_equal(spd.cpu().numpy(), want)
    assert np.array_equal(got.cpu().numpy(), acc)
    assert ctx.get_error() == 0

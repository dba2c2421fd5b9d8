"""The FP64 frame form (a configuration's planes in LDS): AUTO, which takes the
neurons an exchange cannot change from the base pass, against FULL, which
recomputes them all, and against the oracle, at the edges of its frames (the
whole torus, the box of the cone, regions clamped in one direction), of its
tiles (remainders of 0, 2, 4, 8 and 14 sites) and of its workgroup shapes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2204_07816_amd import inputs, nqs

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


def make(net, L, K, C, J2):
    if net == "cnn1":
        w = inputs.cnn1_weights(K, C, 0.05, 31, 1.0)
        return nqs.Context.cnn1(L, 1.0, J2, K, C, w), w, inputs.spins_any(L, 3, 32)
    if net == "cnn2":
        w = inputs.cnn2_weights(K, C, 1.0, 31, 2.0)
        return nqs.Context.cnn2_tj(L, 1.0, 0.4, K, C, w), w, inputs.spins_tj(L, 3, 2 * (L * L // 16), 32)
    w = inputs.stress_weights(K, C, 1.0, 31)
    return nqs.Context(L, 1.0, J2, K, C, w), w, inputs.spins_any(L, 3, 32)


def energies(net, L, K, C, J2, w, sp):
    if net == "cnn1":
        return oracle.cnn1_local_energy(L, 1.0, J2, K, C, w, sp)
    if net == "cnn2":
        return oracle.tj_cnn2_local_energy(L, 1.0, 0.4, K, C, w, sp)
    return oracle.local_energy(L, 1.0, J2, K, C, w, sp)


@pytest.mark.parametrize("net,L,K,C,J2", [
    ("lncosh", 4, 2, 16, 0.5), ("lncosh", 4, 5, 32, 0.5), ("lncosh", 6, 2, 32, 0.0),
    ("lncosh", 8, 2, 16, 0.5), ("lncosh", 10, 4, 16, 0.5), ("lncosh", 12, 6, 32, 0.5),
    ("lncosh", 12, 4, 16, 0.5), ("lncosh", 14, 6, 16, 0.5), ("lncosh", 16, 8, 32, 0.0),
    ("lncosh", 18, 3, 32, 0.5), ("cnn1", 4, 1, 16, 0.5), ("cnn1", 6, 3, 16, 0.0),
    ("cnn1", 10, 6, 16, 0.5), ("cnn1", 12, 2, 16, 0.5), ("cnn1", 14, 4, 16, 0.5),
    ("cnn1", 18, 1, 16, 0.5), ("cnn2", 4, 1, 32, 0.0), ("cnn2", 6, 2, 16, 0.0),
    ("cnn2", 10, 1, 32, 0.0), ("cnn2", 12, 6, 32, 0.0), ("cnn2", 14, 2, 16, 0.0),
])
def test_auto_full_and_oracle(net, L, K, C, J2):
    ctx, w, sp = make(net, L, K, C, J2)
    spd = torch.as_tensor(sp).cuda()
    counts, offs, *_ = ctx.connected(spd)
    n = int(offs[-1])
    full = ctx.log_ratios(spd, mode="full")[:n].cpu().numpy()
    auto = ctx.log_ratios(spd, mode="auto")[:n].cpu().numpy()
    # the same neurons; the two sums over the sites differ by their order, a
    # few roundings of the largest partial sum (64 at most for these sizes)
    f = float(ctx.log_psi(spd)[0].abs().max())
    assert np.max(np.abs(full - auto)) <= 64 * EPS * max(1.0, f)
    ref = energies(net, L, K, C, J2, w, sp)
    for mode in ("full", "auto"):
        e = ctx.local_energy(spd, mode=mode).cpu().numpy()
        assert np.max(np.abs(e - ref)) <= 1e-10 * np.max(np.abs(ref))
    assert ctx.get_error() == 0


def test_several_cache_fills():
    """More samples than one fill of the activation cache holds (4 GiB): each
    sample's energy equals its own call's, bit for bit."""
    L, K, C = 4, 16, 32
    w = inputs.stress_weights(K, C, 1.0, 33)
    sp = torch.as_tensor(inputs.spins_any(L, 512, 34)).cuda()
    B = 73728                      # 15 layers x 16 sites x 32 channels: 61,440 bytes a sample
    big = sp.repeat(B // 512, 1, 1).contiguous()
    ctx = nqs.Context(L, 1.0, 0.5, K, C, w)
    e = ctx.local_energy(big).reshape(-1, 512)
    one = ctx.local_energy(sp)
    assert torch.equal(e, one.expand_as(e))


@pytest.mark.parametrize("L,K,C,B,steps", [
    (4, 2, 16, 5, 7), (4, 2, 16, 3079, 3), (10, 3, 16, 3, 9), (12, 2, 32, 3, 8), (14, 2, 32, 2, 6),
    (18, 2, 16, 2, 6), (20, 2, 16, 2, 5),
])
def test_chains_equal_the_oracle(L, K, C, B, steps):
    """All steps of a chain in one launch, in every workgroup shape: one wave
    per chain (many chains), four, and eight."""
    w = inputs.stress_weights(K, C, 1.0, 41)
    sp = inputs.spins_sz0(L, B, 42)
    rb, ru = inputs.mcmc_randoms(43, 0, steps, B)
    want, acc = oracle.mcmc(L, 1.0, 0.5, K, C, w, sp, rb, ru)
    ctx = nqs.Context(L, 1.0, 0.5, K, C, w)
    spd = torch.as_tensor(sp.copy()).cuda()
    got = ctx.mcmc(spd, torch.as_tensor(rb).cuda(), torch.as_tensor(ru).cuda())
    assert np.array_equal(spd.cpu().numpy(), want)
    assert np.array_equal(got.cpu().numpy(), acc)
    assert ctx.get_error() == 0


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("L,K,C,J2", [
    (4, 2, 16, 0.5), (6, 3, 32, 0.0), (10, 4, 16, 0.5), (12, 5, 32, 0.5), (14, 2, 16, 0.5),
    (16, 6, 32, 0.5), (18, 4, 16, 0.0), (24, 2, 32, 0.5),
])
def test_ratios_equal_the_layered_amplitudes(dtype, L, K, C, J2):
    """Every neuron of the frame form equals the layered kernels' (log_psi) bit
    for bit, so a log ratio is the difference of two of their amplitudes but
    for the order of the FP64 sums over N C terms of size f / (N C): at most
    log2 of the terms' roundings of f in a tree, 64 for a serial order."""
    w = inputs.stress_weights(K, C, 1.0, 51)
    sp = inputs.spins_any(L, 1, 52)
    ctx = nqs.Context(L, 1.0, J2, K, C, w, dtype)
    spd = torch.as_tensor(sp).cuda()
    counts, offs, bonds, _, _ = ctx.connected(spd)
    n = int(offs[-1])
    b = bonds[:n].cpu().numpy()
    dx, dy = np.array([1, 0, 1, 1]), np.array([0, 1, 1, -1])
    i = b >> 2
    x, y = i % L, i // L
    j = (y + dy[b & 3]) % L * L + (x + dx[b & 3]) % L
    pick = np.arange(n) if n <= 400 else np.linspace(0, n - 1, 400).astype(int)
    ex = np.repeat(sp.reshape(1, -1), len(pick), 0)
    r = np.arange(len(pick))
    ex[r, i[pick]], ex[r, j[pick]] = sp.reshape(-1)[j[pick]], sp.reshape(-1)[i[pick]]
    f0 = float(ctx.log_psi(spd)[0][0])
    f1 = ctx.log_psi(torch.as_tensor(ex.reshape(-1, L, L)).cuda())[0].cpu().numpy()
    bound = 64 * EPS * (abs(f0) + np.abs(f1))
    for mode in ("full", "auto"):
        d = ctx.log_ratios(spd, mode=mode)[:n].cpu().numpy()[pick]
        assert np.all(np.abs(d - (f1 - f0)) <= bound)

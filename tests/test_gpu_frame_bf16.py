"""The BF16 frame kernel (a configuration's layers in place in LDS): incremental
and automatic evaluation against the full recomputation, at the edges of its
frames (the whole torus, K + 2 sites wide at least, or the widened box), of its
tiles (1 to 81 of 16 sites, with remainders) and of its dispatch (a wave, four
or eight waves per configuration; the cone kernel from five layers on)."""
import numpy as np
import pytest
import torch

from paper_2204_07816_amd import inputs, nqs

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("L,K,C,B", [
    (4, 2, 32, 1), (4, 2, 32, 40), (4, 2, 16, 40), (6, 4, 16, 9), (6, 4, 32, 20),
    (8, 2, 32, 2), (8, 3, 32, 9), (8, 6, 16, 9), (10, 4, 16, 2), (10, 4, 32, 5),
    (12, 3, 32, 5), (12, 6, 16, 4), (12, 7, 32, 4), (14, 5, 32, 3), (14, 10, 16, 2),
    (16, 4, 32, 2), (16, 9, 16, 2), (18, 12, 16, 1), (20, 8, 16, 2), (24, 3, 16, 1),
    (36, 4, 32, 1), (36, 5, 32, 1), (24, 14, 16, 1),
])
def test_regions_against_full(L, K, C, B):
    w = inputs.stress_weights(K, C, 1.0, 31)
    ctx = nqs.Context(L, 1.0, 0.5, K, C, w, "bf16")
    sp = torch.as_tensor(inputs.spins_any(L, B, 32)).cuda()
    counts, offs, *_ = ctx.connected(sp)
    n = int(offs[-1])
    full = ctx.log_ratios(sp, mode="full")[:n].cpu().numpy()
    # the same neurons; sums over the sites in another order, and with the
    # sites outside the region cancelled: roundings of the largest partial sum
    f = float(ctx.log_psi(sp)[0].abs().max())
    modes = ["auto"]
    if 2 * min(2 + 2 * K + 2, L) ** 2 * (2 * C + 16) <= 159 * 1024:
        modes.append("incremental")
    for mode in modes:
        d = ctx.log_ratios(sp, mode=mode)[:n].cpu().numpy()
        print(L, K, C, B, mode, np.max(np.abs(full - d)), flush=True)
        assert np.max(np.abs(full - d)) <= 64 * EPS * max(1.0, f)
    assert ctx.get_error() == 0


def test_regions_of_several_lattices():
    K, C = 4, 32
    w = inputs.stress_weights(K, C, 1.0, 33)
    ctx = [nqs.Context(L, 1.0, 0.5, K, C, w, "bf16") for L in (6, 8, 12, 16)]
    sps = [torch.as_tensor(inputs.spins_any(c.L, 6, 34)).cuda() for c in ctx]
    es = [torch.empty(6, dtype=torch.float64, device="cuda") for _ in ctx]
    nqs.local_energy_multi(list(zip(ctx, sps, es)))
    for c, sp, e in zip(ctx, sps, es):
        ref = c.local_energy(sp, mode="full").cpu().numpy()
        assert np.max(np.abs(e.cpu().numpy() - ref)) <= 1e-10 * np.max(np.abs(ref))
        assert c.get_error() == 0


@pytest.mark.parametrize("L,K,C", [(6, 2, 16), (8, 3, 32), (10, 8, 16)])
def test_chains_by_regions(L, K, C):
    # more chains than the line below which FULL is kept; decisions against the
    # ratios of the full form
    B, steps = 1100, 3
    w = inputs.stress_weights(K, C, 0.5, 35)
    sp = inputs.spins_any(L, B, 36)
    g = np.random.default_rng(37)
    rb = torch.as_tensor(g.integers(0, 4 * L * L, (steps, B)).astype(np.int32)).cuda()
    ru = torch.as_tensor(g.random((steps, B))).cuda()
    out = []
    for mode in ("auto", "full"):
        ctx = nqs.Context(L, 1.0, 0.5, K, C, w, "bf16")
        s = torch.as_tensor(sp).cuda()
        acc = ctx.mcmc(s, rb, ru, mode=mode)
        out.append((s.cpu().numpy(), acc.cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("L,K,C,B,mode", [(4, 2, 16, 3, "auto"), (14, 3, 16, 70, "auto"),
                                          (12, 6, 32, 40, "incremental"), (8, 5, 32, 40, "full")])
def test_chains_keep_base_pass(L, K, C, B, mode):
    # many steps in one call (the base pass follows the chains that move) against
    # one call a step
    steps = 24
    w = inputs.stress_weights(K, C, 0.3, 45)
    sp = inputs.spins_any(L, B, 46)
    g = np.random.default_rng(47)
    rb = torch.as_tensor(g.integers(0, 4 * L * L, (steps, B)).astype(np.int32)).cuda()
    ru = torch.as_tensor(g.random((steps, B))).cuda()
    ctx = nqs.Context(L, 1.0, 0.5, K, C, w, "bf16")
    one, each = torch.as_tensor(sp).cuda(), torch.as_tensor(sp).cuda()
    acc = ctx.mcmc(one, rb, ru, mode=mode)
    acc2 = torch.zeros_like(acc)
    for t in range(steps):
        ctx.mcmc(each, rb[t:t + 1], ru[t:t + 1], accepted=acc2, mode=mode)
    print(L, K, C, B, mode, "accepted", int(acc.sum()), "of", steps * B, flush=True)
    assert torch.equal(one, each) and torch.equal(acc, acc2)
    assert 0 < int(acc.sum()) < steps * B

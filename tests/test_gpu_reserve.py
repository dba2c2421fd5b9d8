"""Workspace reservations of the frame form: FULL reserves no activation cache,
and AUTO under capture makes do with a reservation for FULL."""
import pytest
import torch

from paper_2204_07816_amd import inputs, nqs

pytestmark = pytest.mark.gpu


def context(net, L, K, C, dtype):
    if net == "cnn2":
        return nqs.Context.cnn2_tj(L, 1.0, 0.4, K, C, inputs.cnn2_weights(K, C, 1.0, 31, 2.0))
    return nqs.Context(L, 1.0, 0.5, K, C, inputs.stress_weights(K, C, 1.0, 31), dtype)


@pytest.mark.parametrize("mode,most", [("full", 700), ("auto", 1500)])
def test_reserved_memory(mode, most):
    """24x24, 12 layers of 32: the cache is 11 planes of 147 KB a sample, 811 MB for
    500; all else is two planes and 12 bytes for each of 2304 pairs a sample."""
    ctx = context("ln", 24, 12, 32, "fp64")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.reserve(500, mode)
    took = (free - torch.cuda.mem_get_info()[0]) / 1e6
    print(mode, took, flush=True)
    assert took < most
    if mode == "auto":
        assert took > 811


@pytest.mark.parametrize("net,L,K,C,dtype", [("ln", 10, 4, 16, "fp64"), ("ln", 12, 5, 32, "fp32"),
                                             ("ln", 10, 4, 8, "fp64"), ("cnn2", 8, 2, 16, "fp64")])
def test_auto_captured_after_reserve_full(net, L, K, C, dtype):
    B = 12
    ctx, plain = context(net, L, K, C, dtype), context(net, L, K, C, dtype)
    sp = torch.as_tensor(inputs.spins_tj(L, B, 8, 32) if net == "cnn2" else inputs.spins_sz0(L, B, 32)).cuda()
    e = torch.empty(B, dtype=torch.float64, device="cuda")
    ctx.reserve(B, "full")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.local_energy(sp, out=e)
    full, auto = plain.local_energy(sp, mode="full"), plain.local_energy(sp)
    for _ in range(3):
        e.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(e, full)
        assert float((e - auto).abs().max()) <= 1e-10 * float(auto.abs().max())
    # eager AUTO on the same context takes regions, the graph stays as it is
    assert torch.equal(ctx.local_energy(sp), auto)
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(e, full)

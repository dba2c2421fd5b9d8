"""The SR solve where its first p.Ap is not positive (here 0: the products
underflow): it stops without an update, in every launch shape and block, and
with nothing left of it for the next solve in the same workspace."""
import pytest
import torch

from paper_2204_07816_amd import inputs
from gpu_helpers import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,K,C,B,odt", [
    (4, 2, 3, 5, "fp64"),             # part of a block
    (4, 5, 11, 130, "fp64"),          # three launches, 18 blocks
    (4, 8, 16, 70, "fp64"),           # past the line for three launches, 65 blocks
    (4, 8, 32, 1100, "fp64"),         # 255 blocks
])
def test_no_update_after_breakdown(L, K, C, B, odt):
    ctx = make_ctx(L, 0.5, K, C, inputs.weights(K, C, 0.1, 91))
    g = torch.Generator(device="cuda")
    g.manual_seed(92)
    O = torch.randn(B, ctx.P, generator=g, device="cuda", dtype=torch.float64)
    e = torch.randn(B, generator=g, device="cuda", dtype=torch.float64)
    ref, rst = (v.clone() for v in ctx.sr_solve(O, e, 1e-2, 7))
    for it in (1, 2, 5):
        # F.F is about 1e-230, u = Obar F about 1e-230, Obar^T u below 1e-324
        x, st = ctx.sr_solve(O * 1e-115, e, 0.0, it)
        assert torch.all(x == 0.0)
        assert float(st[2]) == 1.0 and float(st[3]) == 0.0
        x, st = ctx.sr_solve(O, e, 1e-2, 7)
        assert torch.equal(x, ref) and torch.equal(st, rst)

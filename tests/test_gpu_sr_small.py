"""The launch shapes of the SR solve against each other: the stored-O solve takes
three launches an iteration for few parameters and one, two or four rows a block
by the batch; the solve on recomputed rows takes four launches, and rows by the
chunk.  Every sum has the same order in all of them, so the results are the same
bit for bit."""
import pytest
import torch

from paper_2204_07816_amd import inputs
from gpu_helpers import make_ctx, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,K,C,B,odt", [
    (4, 2, 3, 1, "fp64"), (4, 2, 3, 2, "fp32"),          # P = 114: a part of one block
    (4, 2, 4, 63, "fp32"), (4, 3, 3, 65, "fp64"),        # one and two chunks
    (4, 5, 4, 1024, "fp64"),                             # 16 chunks, two rows a block
    (4, 5, 4, 1025, "fp32"), (4, 2, 3, 2100, "fp64"),    # 17, and 33: four launches
    (4, 8, 16, 130, "fp32"),                             # P = 16,400: past the line
    (4, 7, 16, 130, "fp64"),                             # P = 14,080: below it
])
def test_launch_shapes_agree(L, K, C, B, odt):
    w = inputs.weights(K, C, 0.1, 41)
    sp = to_dev(inputs.spins_sz0(L, B, 42))
    ctx = make_ctx(L, 0.5, K, C, w)
    O = ctx.log_deriv(sp, dtype=odt)
    e = torch.sin(torch.arange(B, dtype=torch.float64, device=sp.device) * 1.7)
    for it in (0, 1, 2, 25):
        x, st = (v.clone() for v in ctx.sr_solve(O, e, 1e-2, it))
        for chunk in (1, 0):
            y, su = ctx.sr_solve_recompute(sp, e, 1e-2, it, dtype=odt, chunk_rows=chunk)
            say(L, K, C, B, odt, "iterations", it, "chunk", chunk, float(st[2]))
            assert torch.equal(x, y) and torch.equal(st, su)
    assert ctx.get_error() == 0

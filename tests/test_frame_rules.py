"""The measured rules of the frame form's dispatch, on the host (no GPU): what
each side of a rule's line was measured to be."""
import host_program

HEAD = r"""
#include <cstdio>
#include "nqs_internal.h"
using namespace nqs;
static nqs_ctx net(int kind, int L, int K, int C, nqs_dtype dt)
{
    nqs_ctx c;
    c.L = L, c.N = L * L, c.K = K, c.C = C, c.net = kind, c.dtype = dt;
    return c;
}
"""


def test_filled_channels_of_short_queues(tmp_path):
    """The layered kernels lead for few channels in short queues: (L, K, C,
    samples) and whether the frame is the faster form there, by at least 7%."""
    cases = [
        (4, 2, 4, 1, 1), (6, 3, 4, 4, 1), (8, 4, 4, 1, 1), (8, 4, 4, 16, 0), (10, 5, 4, 8, 0),
        (16, 4, 4, 1, 0), (16, 4, 4, 2, 0), (16, 4, 4, 4, 1), (20, 2, 4, 4, 1), (24, 4, 4, 2, 1),
        (8, 4, 1, 4, 0), (10, 5, 1, 8, 0), (16, 4, 2, 1, 0), (20, 5, 2, 1, 0), (32, 2, 2, 2, 1),
        (4, 2, 8, 1, 1), (10, 5, 6, 1, 1), (16, 4, 8, 1, 1), (16, 4, 6, 2, 1), (20, 5, 12, 1, 1),
        (28, 3, 3, 1, 1), (20, 2, 1, 1, 0), (28, 3, 1, 1, 0), (32, 2, 1, 4, 1),
    ]
    rows = ",".join("{%d,%d,%d,%d,%d}" % c for c in cases)
    rc, out = host_program.run(tmp_path, HEAD + r"""
int main()
{
    const int t[][5] = {%s};
    int bad = 0;
    for (auto &r : t) {
        const nqs_ctx c = net(kNetLnCosh, r[0], r[1], r[2], NQS_FP64);
        const int64_t cap = (int64_t)4 * c.N * r[3];
        if (frame64_pad_wins(&c, cap) != (r[4] != 0)) {
            ++bad;
            std::printf("L %%d K %%d C %%d B %%d: %%d\n", r[0], r[1], r[2], r[3], !r[4]);
        }
    }
    return bad;
}
""" % rows)
    assert rc == 0, out


def test_chains_of_few_steps(tmp_path):
    """(network, L, K, C, precision, chains, steps, cone) and whether one launch
    for all steps was measured to be the faster form, by at least 5%."""
    ln, c1, c2 = 0, 1, 2
    cases = [
        (ln, 10, 4, 16, 0, 1, 1, 0, 1), (ln, 16, 4, 32, 0, 256, 1, 1, 1), (ln, 24, 4, 16, 0, 1, 1, 1, 0),
        (ln, 24, 4, 16, 0, 16, 8, 1, 1), (ln, 24, 4, 16, 0, 256, 1, 1, 1), (ln, 28, 4, 16, 0, 16, 2, 1, 0),
        (ln, 32, 8, 16, 0, 16, 4, 1, 0), (ln, 32, 8, 16, 0, 256, 1, 1, 1), (ln, 20, 4, 32, 0, 1, 1, 1, 0),
        (ln, 20, 4, 32, 0, 16, 8, 1, 1), (ln, 22, 4, 32, 0, 16, 2, 1, 0), (ln, 24, 6, 32, 0, 1, 4, 1, 0),
        (ln, 24, 6, 32, 0, 64, 8, 1, 1), (ln, 24, 6, 32, 0, 256, 1, 1, 1), (ln, 24, 12, 32, 0, 1, 1, 0, 0),
        (ln, 24, 12, 32, 0, 1, 2, 0, 1), (ln, 30, 12, 16, 0, 1, 1, 0, 0), (ln, 20, 4, 32, 1, 1, 1, 0, 1),
        (ln, 34, 4, 16, 1, 1, 1, 0, 0), (ln, 34, 4, 16, 1, 1, 2, 0, 1), (ln, 30, 2, 16, 1, 16, 1, 0, 0), (ln, 30, 4, 4, 0, 1, 8, 0, 0),
        (ln, 30, 4, 2, 0, 128, 8, 0, 0), (ln, 20, 4, 4, 0, 1, 1, 0, 0), (ln, 20, 4, 4, 0, 1, 8, 0, 1),
        (ln, 30, 2, 8, 0, 1, 1, 0, 0), (ln, 30, 2, 8, 0, 1, 8, 0, 1), (ln, 30, 4, 4, 0, 128, 8, 0, 0),
        (c1, 16, 3, 16, 0, 1, 1, 1, 1), (c1, 28, 2, 16, 0, 1, 2, 1, 0), (c1, 32, 2, 16, 0, 256, 2, 1, 1),
        (c1, 30, 8, 16, 0, 1, 4, 0, 0), (c2, 14, 4, 16, 0, 1, 1, 0, 1), (c2, 28, 2, 16, 0, 64, 2, 0, 1),
        (c2, 22, 6, 32, 0, 1, 1, 0, 0), (c2, 22, 6, 32, 0, 32, 8, 0, 1),
    ]
    rows = ",".join("{%d,%d,%d,%d,%d,%d,%d,%d,%d}" % c for c in cases)
    rc, out = host_program.run(tmp_path, HEAD + r"""
int main()
{
    const int t[][9] = {%s};
    int bad = 0;
    for (auto &r : t) {
        const nqs_ctx c = net(r[0], r[1], r[2], r[3], r[4] ? NQS_FP32 : NQS_FP64);
        if (frame64_chains_pay(&c, r[5], r[6], r[7] != 0) != (r[8] != 0)) {
            ++bad;
            std::printf("net %%d L %%d K %%d C %%d chains %%d steps %%d: %%d\n", r[0], r[1], r[2], r[3],
                        r[5], r[6], !r[8]);
        }
    }
    return bad;
}
""" % rows)
    assert rc == 0, out

"""The frame form's dispatch on the host (no GPU): over every lattice, channel
count, depth, network and precision, a network that it accepts has at most as
many tiles in a layer as the widest workgroup shape forms (eight waves of ten
tiles, split over the 16-channel column blocks), for the base pass, exchanged
configurations and chains."""
import host_program

SOURCE = r"""
#include <cstdio>
#include "nqs_internal.h"
using namespace nqs;
int main()
{
    int accepted = 0, bad = 0;
    for (int net : {kNetLnCosh, kNetCnn1, kNetCnn2})
        for (nqs_dtype dt : {NQS_FP64, NQS_FP32})
            for (int L = 4; L <= 64; L += 2)
                for (int C = 1; C <= 32; ++C)
                    for (int K = 1; K <= 16; ++K) {
                        if (net != kNetLnCosh && dt != NQS_FP64) continue;
                        nqs_ctx c;
                        c.L = L, c.N = L * L, c.K = K, c.C = C, c.net = net, c.dtype = dt;
                        const bool any = frame64_ok(&c) || frame64_pad_ok(&c);
                        if (!any && (frame64_chains_ok(&c) || frame64_pad_chains(&c, 1))) ++bad;
                        if (!any) continue;
                        ++accepted;
                        const int blocks = net == kNetCnn1 || C <= 16 ? 1 : 2;
                        // full tiles of 16 sites; FP64's last four go to a quarter tile
                        const int tiles = (c.N + 15 - (dt == NQS_FP64 ? 4 : 0)) / 16;
                        if (tiles > 8 / blocks * 10) {
                            ++bad;
                            std::printf("net %d dtype %d L %d C %d K %d: %d tiles\n", net, dt, L, C, K, tiles);
                        }
                    }
    std::printf("accepted %d bad %d\n", accepted, bad);
    return bad != 0 || accepted == 0;
}
"""


def test_accepted_networks_fit_the_widest_shape(tmp_path):
    rc, out = host_program.run(tmp_path, SOURCE)
    print(out[-2000:])
    assert rc == 0

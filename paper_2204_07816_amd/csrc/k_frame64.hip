// k_frame64.hip -- host side of the FP64 and FP32 frame form (frame64.h): which
// networks it serves, the frame and workgroup shape of a launch; and the look at
// a sample's zeros outside an item's region (k_frame_zeros).
#include <cmath>

#include "frame64.h"

namespace nqs {

using namespace frame;

namespace {

void launch_any(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape,
                hipStream_t s)
{
    if (c->net == kNetCnn1)
        launch_cnn1(c, a, mode, items, shape, s);
    else if (c->net == kNetCnn2)
        (c->C == 32 ? launch_cnn2_32 : launch_cnn2_16)(c, a, mode, items, shape, s);
    else if (c->dtype == NQS_FP32)
        (frame_ch(c) == 32 ? launch_ln32f : launch_ln16f)(c, a, mode, items, shape, s);
    else
        (frame_ch(c) == 32 ? launch_ln32 : launch_ln16)(c, a, mode, items, shape, s);
}

// The first shape whose waves can form every tile of the largest region at
// once and of which the LDS holds at least eight waves on a CU (two per SIMD).
// A few configurations (of which about half of a queue's room are there) end
// sooner with four waves each: up to four per CU, CNN1, whose waves form both
// column blocks, up to two and a half (one sample: ln cosh 10x10, 4 layers of
// 16, room 400: 82 -> 65 us, 14x14, room 784: 119 -> 107, five 10x10 samples,
// room 2000: 88 -> 94; CNN1 10x10, 6 blocks, 400: 240 -> 166, 6x6, 3 blocks,
// 576: 89 -> 88, 1008: 94 -> 109).
int frame_shape(const nqs_ctx *c, int P, bool regions, int64_t items)
{
    const int C = frame_ch(c);
    const int T = frame_tiles(c, regions);
    const FrameShape *sh = C == 16 ? kShapes16 : kShapes32;
    const int ns = C == 16 ? 4 : 3;
    const int64_t few = (c->net == kNetCnn1 ? 5 : 8) * (int64_t)c->n_cu / 2;
    for (int i = 0; i < ns - 1; ++i) {
        if (c->net == kNetCnn1 && i == 1) continue;      // (not built: two column blocks per wave)
        if (T > frame_room(c, sh[i].W, sh[i].NMAX)) continue;
        if ((int)(kLdsMax / (frame_lds(c, P) * sh[i].PK)) * sh[i].W * sh[i].PK < 8) continue;
        if (sh[i].W == 1 && items < few) continue;
        return i;
    }
    return ns - 1;
}

FrameArgs frame_args(const nqs_ctx *c, const int8_t *spins)
{
    FrameArgs a{};
    a.spins = spins;
    const int C = frame_ch(c);
    const bool pad = C != c->C;
    if (c->dtype == NQS_FP32) {
        const float *w = pad ? c->w_pad32 : c->w_vec32;
        a.w1 = w;
        a.w = w + 10 * C;
    } else if (c->net == kNetLnCosh) {
        const double *w = pad ? c->w_pad64 : c->w_vec64;
        a.w1 = w;
        a.w = w + 10 * C;
    } else if (c->net == kNetCnn1) {
        a.w1 = c->w_canon;
        a.w = c->w_vec64;
    } else {
        a.w1 = c->w_canon;
        a.w = c->w_vec64;
        a.wf = c->w_canon + 3 * C + (int64_t)c->K * (18 * (int64_t)C * C + 2 * C);
    }
    a.err = c->err;
    a.L = c->L;
    a.K = c->K;
    return a;
}

// A sample whose amplitude is 0 (or infinite): a neuron outside an item's region
// (the pair's box widened by S sites) is 0 in S' too, and the ratio undefined as
// in the full recomputation.  A workgroup per sample; others leave at once.
constexpr int kZeroThreads = 64;

__global__ void __launch_bounds__(kZeroThreads)
k_frame_zeros(const uint32_t *__restrict__ queue, const int64_t *__restrict__ offsets, int64_t cap,
              int L, int S, const double *__restrict__ site, const double *__restrict__ f,
              double *__restrict__ dlog)
{
    const int64_t s = blockIdx.x;
    if (isfinite(f[s])) return;
    const int64_t q1 = min(offsets ? offsets[s + 1] : s + 1, cap);
    for (int64_t u = (offsets ? offsets[s] : s) + threadIdx.x; u < q1; u += kZeroThreads) {
        const int b = item_bond(queue[u]), tau = b & 3, x = (b >> 2) % L, y = (b >> 2) / L;
        const int w = (tau == 1 ? 1 : 2) + 2 * S, h = (tau == 0 ? 1 : 2) + 2 * S;
        const int x0 = x - S, y0 = y - S - (tau == 3 ? 1 : 0);
        double v = dlog[u];
        for (int p = 0; p < L * L; ++p) {
            const int dx = ((p % L - x0) % L + L) % L, dy = ((p / L - y0) % L + L) % L;
            if (dx >= w || dy >= h) {
                const double t = site[s * L * L + p];
                v += t - t;
            }
        }
        dlog[u] = v;
    }
}

}  // namespace

void frame64_zeros(const nqs_ctx *c, const uint32_t *queue, const int64_t *offsets, int64_t cap,
                   int64_t B, const double *site, const double *f, double *dlog, hipStream_t s)
{
    if (B <= 0 || cap <= 0) return;
    NQS_LAUNCH(k_frame_zeros, dim3((unsigned)B), dim3(kZeroThreads), 0, s, queue, offsets, cap, c->L,
               frame_reach(c), site, f, dlog);
}

// The torus frame has to fit the LDS and its tiles the widest shape (the base
// pass's, and the last of items and chains): FP32 frames of half the size would
// reach 35x35 sites of 32 channels and 50x50 of 16, but 8 waves hold 40 and 80
// tiles, lattices up to 24x24 and 34x34.
static bool frame_fits(const nqs_ctx *c, bool chains = false)
{
    if (c->dtype != NQS_FP64 && c->dtype != NQS_FP32) return false;
    if (c->net == kNetLnCosh && c->K < 2) return false;
    const FrameShape w = kShapes16[3];
    static_assert(kShapes16[3].W == kShapes32[2].W && kShapes16[3].NMAX == kShapes32[2].NMAX,
                  "one widest shape");
    return frame_lds(c, c->L, chains) <= kLdsMax && frame_tiles(c, false) <= frame_room(c, w.W, w.NMAX);
}

bool frame64_ok(const nqs_ctx *c)
{
    if (c->net == kNetCnn1 ? c->C != 16 : (c->C != 16 && c->C != 32)) return false;
    return frame_fits(c);
}

bool frame64_pad_ok(const nqs_ctx *c)
{
    return c->net == kNetLnCosh && c->C < 32 && c->C != 16 && frame_fits(c);
}

// The vector path costs about 1.1e-5 us per channel for each site and layer of
// a configuration (FP32 0.7e-5), the frame 1.2e-4 us for each that it forms
// again, whatever the channels: it leads where the region is less than that
// share of the lattice (FP64, 8 channels: 24x24, 5 layers, share 0.12: 17.9 ->
// 4.6 ms; 10x10, 4 layers, 0.54: 7.1 -> 5.0 ms; 4 channels, 6x6, 2 layers,
// 0.72: 0.31 against 0.50 ms).  Short queues are bound by launches, of which
// the frame needs two, and by the latency of one configuration, which the
// frame's 16 channels cost whatever C is: from five channels on it leads (one
// sample, 10x10, 5 layers of 8: 160 -> 78 us; 16x16, 4 layers of 6: 171 -> 96),
// with three or four on small lattices only (room 256 of 8x8, 4 layers of 4: 69
// -> 57 us, 4096: 86 against 105; one sample of 16x16: 80 against 94), and with
// few channels the share's rule holds from a queue of some length on (16x16, 4
// layers of 4, room 2048: 97 against 115 us, 4096: 145 -> 115).
bool frame64_pad_wins(const nqs_ctx *c, int64_t cap)
{
    const int64_t cu = c->n_cu;
    const int64_t room = c->C >= 5 || (c->C >= 3 && c->N <= 16) ? 16 : (c->C >= 3 && c->N <= 100 ? 4 : 0);
    if (cap <= room * cu) return true;
    if (c->C <= 4 && cap * c->C < 36 * cu) return false;
    double inc = 0.0;
    for (int l = 1; l <= c->K; ++l) {
        const double e = std::min(2 + 2 * l, c->L);
        inc += e * e;
    }
    return inc < (c->dtype == NQS_FP32 ? 0.06 : 0.09) * c->C * c->K * c->N;
}

bool frame64_suits(const nqs_ctx *c)
{
    return frame_shape(c, std::min(c->L, 2 * frame_reach(c) + 4), true, INT64_MAX) < 3;
}

bool cone64_ok(const nqs_ctx *c)
{
    return c->dtype == NQS_FP64 && c->net == kNetLnCosh && (c->C == 16 || c->C == 32) &&
           c->K >= 2 && c->K <= 8 && c->L >= 2 * c->K + 4;
}

int64_t frame64_slots(const nqs_ctx *c)
{
    return c->net == kNetLnCosh ? c->K - 1 : (c->net == kNetCnn1 ? 2 * c->K - 1 : 2 * c->K);
}

size_t frame64_cache_bytes(const nqs_ctx *c, int64_t cB)
{
    return (c->dtype == NQS_FP32 ? sizeof(float) : sizeof(double)) * (size_t)frame64_slots(c) * (size_t)cB * c->N * frame_ch(c);
}

// samples per cache fill: at most 16 GiB of cached activations
int64_t cone64_chunk(const nqs_ctx *c, int64_t B)
{
    const int64_t m = (int64_t)(((size_t)16 << 30) / std::max<size_t>(frame64_cache_bytes(c, 1), 1));
    return std::max<int64_t>(1, std::min(m, std::max<int64_t>(B, 1)));
}

void frame64_base(const nqs_ctx *c, const int8_t *spins, int64_t cB, int64_t b0, int64_t nb,
                  void *cache, double *site, int32_t *neg, double *f, int8_t *sgn, hipStream_t s)
{
    if (nb <= 0) return;
    FrameArgs a = frame_args(c, spins);
    a.cache = cache;
    a.site = site;
    a.neg = neg;
    a.f = f;
    a.sgn = sgn;
    a.cB = cB;
    a.b0 = b0;
    a.nb = nb;
    a.P = c->L;
    launch_any(c, a, kBase, nb, 0, s);
}

void frame64_conn(const nqs_ctx *c, const int8_t *spins, const uint32_t *queue,
                  const int64_t *offsets, int64_t cap, int64_t cB, int64_t b0, int64_t nb,
                  const void *cache, const double *site, const int32_t *neg, double *dlog,
                  int8_t *isign, hipStream_t s)
{
    if (nb <= 0 || cap <= 0) return;
    FrameArgs a = frame_args(c, spins);
    a.queue = queue;
    a.offsets = offsets;
    a.cap = cap;
    a.cache = const_cast<void *>(cache);
    a.site = const_cast<double *>(site);
    a.neg = const_cast<int32_t *>(neg);
    a.cB = cB;
    a.b0 = b0;
    a.nb = nb;
    a.dlog = dlog;
    a.isign = isign;
    a.F = frame_reach(c) + 1;
    a.regions = cache ? 1 : 0;
    a.P = cache ? std::min(c->L, 2 * a.F + 2) : c->L;
    const int64_t items = offsets ? cap : nb;
    launch_any(c, a, kItems, items, frame_shape(c, a.P, cache != nullptr, items), s);
}

bool frame64_chains_ok(const nqs_ctx *c)
{
    return frame64_ok(c) && frame_fits(c, true);
}

// A launch per chain and not per layer and step pays for networks with filled
// channels until the chains fill the chip several times (6x6, 3 layers of 4, 32
// steps of 1024 chains: 1.61 -> 0.51 ms).
bool frame64_pad_chains(const nqs_ctx *c, int64_t B)
{
    return frame64_pad_ok(c) && frame_fits(c, true) &&
           (B <= (int64_t)8 * c->n_cu || frame64_pad_wins(c, B));
}

// A call of n steps is n + 1 evaluations of the torus by the one CU that holds
// a chain (the first gives the terms of its configuration).  Step by step, few
// chains are spread over the whole chip, in a time that hardly depends on the
// lattice; `grown` is how it has grown at B chains (32x32, 8 layers of 16: 1, 64
// and 256 chains 209, 255, 540 us; 20x20, 4 layers of 32: 182, 212, 295).
// `share` is the time of one evaluation against such a step, fitted to FP64
// measurements of few chains (us of a step, 1, 2, 4 and 8 steps a call, against
// step by step):
//   16 channels, 4 layers: 20x20 103 73 57 48 / 92; 30x30 181 131 106 94 / 97
//   32 channels, 4 layers: 16x16 164 122 99 86 / 168; 22x22 290 213 175 155 / 180
//   CNN1, 3 blocks: 16x16 108 77 61 54 / 130; 20x20 166 120 98 86 / 140
// The step-by-step form costs half as much again without a cone, almost twice
// as much in FP32, and with 3 or 4 and fewer channels less than with 16.
bool frame64_chains_pay(const nqs_ctx *c, int64_t B, int n_steps, bool cone)
{
    const bool wide = frame_ch(c) == 32, pad = frame_ch(c) != c->C;
    const double fill = (double)B / std::max(c->n_cu, 1);
    const double grown = 1.0 + (c->C <= 4 ? 0.75 : 1.5) * c->N / 1024 * fill * std::sqrt(fill);
    double share = wide ? (c->N + 150) / 820.0 : (c->N + 180) / 1150.0;
    if (c->net == kNetCnn1)
        share = (c->N + 250) / 1250.0 * (cone ? 1.0 : 0.92);
    else if (c->net == kNetCnn2)
        share *= wide ? 0.83 : 0.74;
    else if (pad)
        share *= wide ? 0.92 : (c->C >= 5 ? 0.8 : (c->C >= 3 ? 1.45 : 2.0));
    else if (c->dtype == NQS_FP32)
        share *= 0.55;
    else if (!cone)
        share *= 0.68;
    return (n_steps + 1.0) * share <= n_steps * grown;
}

void frame64_chains(const nqs_ctx *c, int8_t *spins, int64_t B, int n_steps, const uint32_t *rnd,
                    const double *un, int32_t *accepted, hipStream_t s)
{
    if (B <= 0 || n_steps <= 0) return;
    FrameArgs a = frame_args(c, spins);
    a.chains = spins;
    a.rnd = rnd;
    a.un = un;
    a.accepted = accepted;
    a.B = a.nb = B;
    a.n_steps = n_steps;
    a.j1 = nn_moves(c) ? 1 : 0;
    a.j2 = nnn_moves(c) ? 1 : 0;
    a.P = c->L;
    // A chain is a serial run of steps: four waves share each (10x10, 4 layers
    // of 16, 32 steps of 512 chains: 0.65 ms against 1.17 for one wave and 0.82
    // for eight) while their tiles allow; one wave each where the chains alone
    // fill three waves per SIMD (4096 chains: 3.25 against 3.54 ms).
    const int T = frame_tiles(c, false);
    auto holds = [&](const FrameShape &s) { return T <= frame_room(c, s.W, s.NMAX); };
    const int C = frame_ch(c);
    int shape = 3;
    if (C == 16 && holds(kShapes16[0]) && B >= 12 * (int64_t)c->n_cu)
        shape = 0;
    else if (C == 16 && holds(kShapes16[2]))
        shape = 2;
    else if (C == 32 && holds(kShapes32[0]))
        shape = 0;
    launch_any(c, a, kChains, B, shape, s);
}

}  // namespace nqs

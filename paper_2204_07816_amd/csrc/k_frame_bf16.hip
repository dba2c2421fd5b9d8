// k_frame_bf16.hip -- the exchanged-configuration pass of the BF16 form where
// the cone kernel (k_net_cone.hip: 32 channels, 5 layers and more in windows
// that do not wrap) is not taken: windows that wrap around the torus, 16
// channels, or few layers [Sec. 5.4.1].
//
// A configuration's layers run in place on a frame of P x P sites in LDS, the
// whole torus (P = L) or the exchanged pair's box widened by K + 1.  Layer k is
// formed on R_k, the box widened by k sites (clamped to the torus); the ring
// R_{k+2} \ R_k comes from the base pass's cached activations.  These lattices
// have 3 to 9 tiles of 16 sites per layer, so a workgroup per configuration
// spends its time between the tiles: in each wave's fetch of the layer's
// weights, and in barriers (12x12, 6 layers of 32 channels: matrix cores 13%
// busy, 5.4 ms for 178,600 configurations).  Here one wave takes a
// configuration by itself while its tiles fit the registers: it forms all
// tiles of a layer at once, so the weights of a tap are fetched once per
// configuration, and it has no barrier; three waves per SIMD cover the
// latencies.  Larger regions are shared by four or eight waves.
// Same case here: 3.1 ms.  What bounds it now is the vector unit: ln cosh is
// about 14 instructions and two quarter-rate ones per value.
//
// The frame is kept as planes of 16-byte chunks (8 channels), an odd number of
// chunks apart: the 16 sites of a lane group's operand are 256 contiguous bytes.
// Every value is formed as in the base pass (mfma_common.h), so sites that the
// exchange does not reach cancel exactly.
#include <algorithm>
#include <type_traits>

#include "mfma_common.h"

namespace nqs {
namespace {

using mf::bf16x8;
using mf::floatx4;
using mf::Shape;

constexpr int kXcd = 8;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct BfJob {
    const int8_t *spins;
    const uint32_t *queue;
    const int64_t *qlen;
    int64_t capacity;
    const bf16x8 *wa;           // layers 2..K: [KS][NH][64] operands each
    const float *w1, *bias;
    const uint16_t *cache;      // [B][K-1][N][C]
    const double *hsum;         // [B][N]
    double *dlog;
    int32_t *err;
    int L, K, P;
};

// Up to kMaxConnJobs lattices (contexts of one network shape) in one launch:
// their queue items form one index space, job after job.
struct BfJobs {
    BfJob job[kMaxConnJobs];
    int n;
    int lds;                    // LDS bytes of one configuration (the largest job's)
};

__device__ inline int wrap1(int a, int P) { return a < 0 ? a + P : (a >= P ? a - P : a); }
__host__ __device__ inline int plane_bytes16(int P) { return ((P * P) | 1) * 16; }

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    return (uint32_t)mf::to_bf16(a) | ((uint32_t)mf::to_bf16(b) << 16);
}

struct Region {
    int x0, y0, w, h;
};

// this lane's site of a tile: its byte offset in the lane group's plane, byte
// steps to the neighbours
struct TileSite {
    int org, up, dn, lf, rt;
};

// tiles whose accumulators a wave holds at once (a layer with more takes two
// or three passes over its weights)
constexpr int kPart = 5;

// Accumulators of N tiles (the last formed only when `last`): bias, then the
// K-steps in the base pass's order.  32 channels: a K-step is a tap.  16
// channels: two taps, lane groups 0-1 the first, 2-3 the second (clamped to
// tap 8, whose partner's weights are zero).  The next K-step's weights are
// fetched while this one's MFMAs issue.
template <int C, int N>
__device__ __forceinline__ void conv_tiles(const unsigned char *fr, bool last,
                                           const TileSite (&st)[N], const bf16x8 *wl, int g,
                                           const float (&bias)[Shape<C>::NH][4],
                                           floatx4 (&acc)[N][Shape<C>::NH])
{
    using S = Shape<C>;
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
        for (int hh = 0; hh < S::NH; ++hh)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[t][hh][r] = bias[hh][r];
    bf16x8 wv[S::NH], wn[S::NH];
#pragma unroll
    for (int hh = 0; hh < S::NH; ++hh) wv[hh] = wl[hh * 64];
    auto step = [&](int j, auto &&at) {
        // (the last step fetches step 0's again, unused)
        const bf16x8 *wp = wl + (j + 1 < S::KS ? (j + 1) * S::NH * 64 : 0);
#pragma unroll
        for (int hh = 0; hh < S::NH; ++hh) wn[hh] = wp[hh * 64];
#pragma unroll
        for (int t = 0; t < N; ++t) {
            if (t + 1 < N || last) {
                const bf16x8 bv = *(const bf16x8 *)(fr + at(t));
#pragma unroll
                for (int hh = 0; hh < S::NH; ++hh)
                    acc[t][hh] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[hh], bv, acc[t][hh],
                                                                        0, 0, 0);
            }
        }
#pragma unroll
        for (int hh = 0; hh < S::NH; ++hh) wv[hh] = wn[hh];
    };
    if constexpr (C == 32) {
#pragma unroll 1
        for (int ty = 0; ty < 3; ++ty) {
            int row[N];
#pragma unroll
            for (int t = 0; t < N; ++t)
                row[t] = st[t].org + (ty == 0 ? st[t].up : (ty == 2 ? st[t].dn : 0));
#pragma unroll
            for (int tx = 0; tx < 3; ++tx)
                step(3 * ty + tx, [&](int t) {
                    return row[t] + (tx == 0 ? st[t].lf : (tx == 2 ? st[t].rt : 0));
                });
        }
    } else {
        auto tap = [&](const TileSite &s, int t) {
            return (t / 3 == 0 ? s.up : (t / 3 == 2 ? s.dn : 0)) + (t % 3 == 0 ? s.lf : (t % 3 == 2 ? s.rt : 0));
        };
#pragma unroll
        for (int j = 0; j < S::KS; ++j)
            step(j, [&](int t) {
                const int ta = 2 * j, tb = 2 * j + 1 > 8 ? 8 : 2 * j + 1;
                return st[t].org + ((g >> 1) ? tap(st[t], tb) : tap(st[t], ta));
            });
    }
}

// f(integral_constant n) for a run-time 1 <= n <= N
template <int N, class Fn>
__device__ __forceinline__ void with_count(int n, Fn &&f)
{
    if constexpr (N > 1)
        if (n < N) return with_count<N - 1>(n, f);
    f(std::integral_constant<int, N>{});
}

// W waves form a configuration; PK > 1 (W = 1 only): PK waves of a workgroup,
// each with its own configurations and no barrier between them
template <int C, int W, int PK, int NMAX, int EU, bool FEW>
__global__ void __launch_bounds__(W * PK * 64, EU)
k_frame_bf16(BfJobs jobs)
{
    static_assert(PK == 1 || W == 1, "only single waves share a workgroup");
    using S = Shape<C>;
    constexpr int NT = W * 64, CHK = S::CHUNKS;
    auto sync = [] {
        if constexpr (W == 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr bool PARTS = W == 4 || FEW;            // more waves than one for up to 24 tiles
    __shared__ double red[W == 8 ? W : 1];
    double *terms = (double *)(lds + jobs.lds);      // PARTS: [tiles][16] of the last layer
    const int pk = PK > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    unsigned char *fr = lds + pk * jobs.lds;
    const int tid = PK > 1 ? threadIdx.x & 63 : threadIdx.x, lane = tid & 63;
    const int wave = PK > 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n16 = lane & 15;

    // first item of each job in the common index space
    int64_t first[kMaxConnJobs + 1];
    first[0] = 0;
#pragma unroll
    for (int j = 0; j < kMaxConnJobs; ++j)
        first[j + 1] = first[j] + (j < jobs.n ? min(jobs.job[j].qlen[0], jobs.job[j].capacity) : 0);
    const int64_t n_units = first[kMaxConnJobs];
    // XCD-contiguous ranges of the queue: consecutive items (mostly of one
    // sample) stay on one XCD, whose L2 then serves that sample's cache
    const int xcd = blockIdx.x % kXcd;
    const int64_t seg = (n_units + kXcd - 1) / kXcd;
    const int64_t u_end = min(n_units, (xcd + 1) * seg);
    const int64_t u_step = (int64_t)(gridDim.x / kXcd) * PK;
    int w1_job = -1;            // job whose layer-1 weights are in LDS (the frames differ in size)
    for (int64_t u = xcd * seg + (int64_t)(blockIdx.x / kXcd) * PK + pk; u < u_end; u += u_step) {
        int jb = 0;
        int64_t u0 = 0;
#pragma unroll
        for (int j = 1; j < kMaxConnJobs; ++j)
            if (u >= first[j]) jb = j, u0 = first[j];
        const BfJob &a = jobs.job[jb];
        const int64_t unit = u - u0;
        const int L = a.L, N0 = L * L, P = a.P, K = a.K, F = K + 1;
        const bool torus = P == L;
        const int SB = plane_bytes16(P);
        float *w1s = (float *)(fr + CHK * SB);       // layer 1: [9 taps, bias][C], slot order
        int8_t *sf = (int8_t *)(w1s + 10 * C);
        if (jb != w1_job) {
            for (int q = tid; q < 10 * C; q += NT) {
                const int ch = mf::chan_of_slot<C>(q % C);
                w1s[q] = q < 9 * C ? a.w1[q / C * C + ch] : a.bias[ch];
            }
            w1_job = jb;
        }
        const uint32_t e = a.queue[unit];
        const int s = item_sample(e), b = item_bond(e), tau = b & 3, i0 = b >> 2;
        const int xi = i0 % L, yi = i0 / L;
        const int qi = i0, qj = wrap1(yi + bond_dy(tau), L) * L + wrap1(xi + bond_dx(tau), L);
        const int ax = xi, ay = (tau == 3) ? wrap1(yi - 1, L) : yi;
        const int w0 = (tau == 1) ? 1 : 2, h0 = (tau == 0) ? 1 : 2;
        const uint16_t *cache_s = a.cache + (int64_t)s * (K - 1) * N0 * C;
        auto region = [&](int k) {
            Region r{0, 0, L, L};
            if (w0 + 2 * k < L) r.x0 = torus ? wrap1(ax - k, L) : F - k, r.w = w0 + 2 * k;
            if (h0 + 2 * k < L) r.y0 = torus ? wrap1(ay - k, L) : F - k, r.h = h0 + 2 * k;
            return r;
        };
        // lattice coordinate of a frame coordinate; a torus frame is the lattice
        auto lat = [&](int f, int anchor) { return torus ? f : wrap1(anchor - F + f, L); };
        auto inside = [&](int f) { return f >= P ? f - P : f; };

        // the exchanged configuration on R_1 and one site around it, row by row
        const Region r1 = region(1);
        const int sw = r1.w + 2, sn = sw * (r1.h + 2);
        const uint32_t smul = ((1u << 20) + sw - 1) / sw;
        for (int q = tid; q < sn; q += NT) {
            const int v = (int)(((uint32_t)q * smul) >> 20);
            const int fx = wrap1(r1.x0 + q - v * sw - 1, P), fy = wrap1(r1.y0 + v - 1, P);
            int site = lat(fy, ay) * L + lat(fx, ax);
            site = (site == qi) ? qj : ((site == qj) ? qi : site);
            sf[q] = a.spins[(int64_t)s * N0 + site];
        }
        sync();
        // ring R_{k+2} \ R_k from the sample's activations of layer k.  Few
        // configurations (FEW) wait for each round of loads, so the whole ring
        // is one or two: the rows beyond R_k, then the columns beside it (14x14,
        // 5 layers of 16, 357 configurations: 21.6 us by rows, 16.4 so).
        auto ring_once = [&](int k) {
            const Region in = region(k), out = region(k + 2);
            const int eh = out.h - in.h, ew = out.w - in.w;
            const int nrow = eh * out.w, total = (nrow + ew * in.h) * CHK;
            // beyond R_k's end first, two where the ring has two sides
            const int hb = out.h == P ? eh : 2, wb = out.w == P ? ew : 2;
            const uint32_t mw = ((1u << 20) + out.w - 1) / out.w, me = ew ? ((1u << 20) + ew - 1) / ew : 0;
            const uint16_t *src = cache_s + (int64_t)(k - 1) * N0 * C + 8 * (tid % CHK);
            auto entry = [&](int q, int &f) {
                const int e = (q < total ? q : 0) / CHK;
                int fx, fy;
                if (e < nrow) {
                    const int v = (int)(((uint32_t)e * mw) >> 20);
                    fy = v < hb ? inside(in.y0 + in.h + v) : inside(out.y0 + v - hb);
                    fx = inside(out.x0 + e - v * out.w);
                } else {
                    const int v = (int)(((uint32_t)(e - nrow) * me) >> 20), h = e - nrow - v * ew;
                    fy = inside(in.y0 + v);
                    fx = h < wb ? inside(in.x0 + in.w + h) : inside(out.x0 + h - wb);
                }
                f = (fy * P + fx) * 16 + (tid % CHK) * SB;
                return *(const u32x4 *)(src + (lat(fy, ay) * L + lat(fx, ax)) * C);
            };
            for (int q = tid; q < total; q += 2 * NT) {       // (NT is a multiple of CHK)
                int f0, f1;
                const u32x4 d0 = entry(q, f0), d1 = entry(q + NT, f1);
                *(u32x4 *)(fr + f0) = d0;
                if (q + NT < total) *(u32x4 *)(fr + f1) = d1;
            }
        };
        // layer 1 on R_1 (vector ALU): thread (site, lane group's channels)
        {
            const uint32_t mul = ((1u << 20) + r1.w - 1) / r1.w;
            for (int q = tid; q < r1.w * r1.h * 4; q += NT) {
                const int p = q >> 2, gg = q & 3;
                const int v = (int)(((uint32_t)p * mul) >> 20), x = p - v * r1.w;
                float sv[9];
#pragma unroll
                for (int t = 0; t < 9; ++t) sv[t] = (float)sf[(v + t / 3) * sw + x + t % 3];
                // layer1_z's order (bias, then the taps) for this group's channels
                float z[S::CG], h[S::CG];
#pragma unroll
                for (int i = 0; i < S::CG; ++i) z[i] = w1s[9 * C + gg * S::CG + i];
#pragma unroll
                for (int t = 0; t < 9; ++t)
#pragma unroll
                    for (int i = 0; i < S::CG; ++i)
                        z[i] = __builtin_fmaf(w1s[t * C + gg * S::CG + i], sv[t], z[i]);
                mf::ln_cosh_n<S::CG>(z, h);
                uint32_t w[S::CG / 2];
#pragma unroll
                for (int i = 0; i < S::CG / 2; ++i) w[i] = pack2(h[2 * i], h[2 * i + 1]);
                unsigned char *to = fr + (inside(r1.y0 + v) * P + inside(r1.x0 + x)) * 16;
                if constexpr (C == 32)
                    *(u32x4 *)(to + gg * SB) = (u32x4){w[0], w[1], w[2], w[3]};
                else
                    *(uint2 *)(to + (gg >> 1) * SB + (gg & 1) * 8) = uint2{w[0], w[1]};
            }
        }
        // the ring where configurations are many: the threads span a stretch of a row
        // (site, chunk), the rows are taken four at a time
        auto ring_rows = [&](int k) {
            constexpr int XP = NT / CHK;
            const Region in = region(k), out = region(k + 2);
            if (in.w == out.w && in.h == out.h) return;
            const uint16_t *src = cache_s + (int64_t)(k - 1) * N0 * C;
            const int c = tid % CHK;
            for (int xb = 0; xb < out.w; xb += XP) {
                const int x = xb + tid / CHK;
                const int fx = inside(out.x0 + min(x, out.w - 1));
                const int dx = fx - in.x0 + (fx < in.x0 ? P : 0);
                const bool side = x < out.w && dx >= in.w, live = x < out.w;
                const uint16_t *gx = src + lat(fx, ax) * C + 8 * c;
                unsigned char *fc = fr + c * SB + fx * 16;
                auto row = [&](int v, bool &on) {
                    const int fy = inside(out.y0 + min(v, out.h - 1));
                    const int dy = fy - in.y0 + (fy < in.y0 ? P : 0);
                    on = v < out.h && (dy >= in.h ? live : side);
                    return fy;
                };
                auto get = [&](int fy, bool on) {
                    return *(const u32x4 *)(gx + (on ? lat(fy, ay) * L * C : 0));
                };
                for (int v = 0; v < out.h; v += 4) {
                    bool o0, o1, o2, o3;
                    const int f0 = row(v, o0), f1 = row(v + 1, o1), f2 = row(v + 2, o2), f3 = row(v + 3, o3);
                    if (__ballot(o0 || o1 || o2 || o3) == 0) continue;
                    const u32x4 d0 = get(f0, o0), d1 = get(f1, o1), d2 = get(f2, o2), d3 = get(f3, o3);
                    if (o0) *(u32x4 *)(fc + f0 * P * 16) = d0;
                    if (o1) *(u32x4 *)(fc + f1 * P * 16) = d1;
                    if (o2) *(u32x4 *)(fc + f2 * P * 16) = d2;
                    if (o3) *(u32x4 *)(fc + f3 * P * 16) = d3;
                }
            }
        };
        auto ring = [&](int k) {
            if constexpr (FEW) ring_once(k);
            else ring_rows(k);
        };
        ring(1);
        sync();

        // Last layer: one wave and several give the same sum, since the choice
        // depends on the launch's other configurations.  The one wave adds its lanes'
        // tiles in order, then the lanes in a tree; of several, the first does so
        // from LDS (up to 24 tiles; beyond, always eight waves, each for itself).
        double fsum = 0.0;
        for (int k = 2; k <= K; ++k) {
            const Region r = region(k);
            const int nl = r.w * r.h, T = (nl + 15) >> 4;
            const uint32_t mul = ((1u << 20) + r.w - 1) / r.w;
            float bias[S::NH][4];
#pragma unroll
            for (int hh = 0; hh < S::NH; ++hh)
#pragma unroll
                for (int i = 0; i < 4; ++i) bias[hh][i] = a.bias[(k - 1) * C + 16 * hh + 4 * g + i];
            const bf16x8 *wl = a.wa + (int64_t)(k - 2) * S::KS * S::NH * 64 + lane;
            // tiles wave + W t; the workgroup's largest count is the compiled
            // one, and a wave with one less skips the last
            with_count<NMAX>((T + W - 1) / W, [&](auto count) {
                constexpr int TN = decltype(count)::value;
                // at most kPart tiles hold accumulators at a time; the packed
                // results of all wait until every tile has read the frame
                constexpr int NP = (TN + kPart - 1) / kPart;
                constexpr int N1 = (TN + NP - 1) / NP;
                const bool last = wave + W * (TN - 1) < T;
                uint32_t out[TN][S::CG / 2];
                int to[TN];
                auto part = [&](auto first_tile, auto tiles) {
                    constexpr int T0 = decltype(first_tile)::value, N = decltype(tiles)::value;
                    const bool full = T0 + N < TN || last;
                    TileSite st[N];
#pragma unroll
                    for (int t = 0; t < N; ++t) {
                        const int q = (wave + W * (T0 + t)) * 16 + n16, p = min(q, nl - 1);
                        const int v = (int)(((uint32_t)p * mul) >> 20);
                        const int fx = inside(r.x0 + p - v * r.w), fy = inside(r.y0 + v), f = fy * P + fx;
                        st[t].org = f * 16 + (C == 32 ? g : (g & 1)) * SB;
                        to[T0 + t] = (q < nl ? f : P * P) * 16;     // past the end: the spare chunk
                        st[t].up = (fy == 0 ? P - 1 : -1) * P * 16;
                        st[t].dn = (fy == P - 1 ? 1 - P : 1) * P * 16;
                        st[t].lf = (fx == 0 ? P - 1 : -1) * 16;
                        st[t].rt = (fx == P - 1 ? 1 - P : 1) * 16;
                    }
                    floatx4 acc[N][S::NH];
                    conv_tiles<C, N>(fr, full, st, wl, g, bias, acc);
#pragma unroll
                    for (int t = 0; t < N; ++t) {
                        if (t + 1 == N && !full) break;
                        float zv[S::CG], hv[S::CG];
#pragma unroll
                        for (int i = 0; i < S::CG; ++i) zv[i] = acc[t][i >> 2][i & 3];
                        mf::ln_cosh_n<S::CG>(zv, hv);
                        if (k < K) {
#pragma unroll
                            for (int i = 0; i < S::CG / 2; ++i)
                                out[T0 + t][i] = pack2(hv[2 * i], hv[2 * i + 1]);
                        } else {
                            // the site's channel sum (as the base pass takes it)
                            // less the sample's
                            double sum = 0.0;
#pragma unroll
                            for (int i = 0; i < S::CG; ++i) sum += (double)hv[i];
                            sum += __shfl_xor(sum, 16);
                            sum += __shfl_xor(sum, 32);
                            const int f = to[T0 + t] >> 4, fy = f / P;
                            double d = 0.0;
                            if (g == 0 && f < P * P)
                                d = sum - a.hsum[(int64_t)s * N0 + lat(fy, ay) * L + lat(f - fy * P, ax)];
                            if constexpr (!PARTS)
                                fsum += d;
                            else if (g == 0)
                                terms[(wave + W * (T0 + t)) * 16 + n16] = d;
                        }
                    }
                };
                part(std::integral_constant<int, 0>{}, std::integral_constant<int, N1>{});
                if constexpr (NP >= 2)
                    part(std::integral_constant<int, N1>{},
                         std::integral_constant<int, (TN - N1 < N1 ? TN - N1 : N1)>{});
                if constexpr (NP >= 3)
                    part(std::integral_constant<int, 2 * N1>{},
                         std::integral_constant<int, (TN - 2 * N1 < N1 ? TN - 2 * N1 : N1)>{});
                if constexpr (NP >= 4)
                    part(std::integral_constant<int, 3 * N1>{}, std::integral_constant<int, TN - 3 * N1>{});
                if (k == K) return;
                sync();                      // every read of the frame for layer k is done
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    if (t + 1 < TN || last) {
                        unsigned char *p = fr + to[t];
                        if constexpr (C == 32)
                            *(u32x4 *)(p + g * SB) = (u32x4){out[t][0], out[t][1], out[t][2], out[t][3]};
                        else
                            *(uint2 *)(p + (g >> 1) * SB + (g & 1) * 8) = uint2{out[t][0], out[t][1]};
                    }
            });
            if (k < K) ring(k);
            sync();
        }

        if constexpr (PARTS) {
            const Region r = region(K);
            const int T = (r.w * r.h + 15) >> 4;
            if (tid < 16)
#pragma unroll 4
                for (int t = 0; t < T; ++t) fsum += terms[t * 16 + tid];
        }
        if (!PARTS || wave == 0)
            for (int off = 32; off > 0; off >>= 1) fsum += __shfl_xor(fsum, off);
        if constexpr (W == 8 && !PARTS) {
            if (lane == 0) red[wave] = fsum;
            __syncthreads();
            fsum = 0.0;
            for (int w = 0; w < W; ++w) fsum += red[w];
        }
        if (tid == 0) {
            if (!isfinite(fsum)) atomicOr(a.err, kErrNonFinite);
            a.dlog[unit] = fsum;
        }
    }
}

constexpr size_t kLdsMax = 160 * 1024 - 512;

int frame_side(const nqs_ctx *c) { return std::min(c->L, 2 * c->K + 4); }

size_t frame_bytes(const nqs_ctx *c)
{
    const int P = frame_side(c);
    return ((size_t)(c->C / 8) * plane_bytes16(P) + 40 * c->C + (size_t)(P + 2) * (P + 2) + 15) &
           ~(size_t)15;
}

template <int C, int W, int PK, int NMAX, int EU, bool FEW = false>
void launch_w(const BfJobs &jobs, int n_cu, int64_t items, hipStream_t s)
{
    const auto kernel = k_frame_bf16<C, W, PK, NMAX, EU, FEW>;
    const int lds = jobs.lds * PK + (W == 4 || FEW ? W * NMAX * 16 * (int)sizeof(double) : 0);
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    int occ = 1;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, W * PK * 64, lds);
    int64_t grid = std::min((int64_t)std::max(occ, 1) * n_cu, (items + PK - 1) / PK);
    grid = std::max<int64_t>(kXcd, (grid + kXcd - 1) / kXcd * kXcd);
    NQS_LAUNCH(kernel, dim3((unsigned)grid), dim3(W * PK * 64), lds, s, jobs);
}

}  // namespace

// the lattices served: two windows of the largest layer, as padded sites, fit
// the LDS (the frame is smaller)
bool mfma_inc_supported(const nqs_ctx *c)
{
    const int e = std::min(2 + 2 * c->K + 2, c->L);
    return mfma_supported(c) && c->L >= c->K + 2 &&
           2 * (size_t)(e * e) * (c->C * 2 + 16) <= 160 * 1024 - 1024;
}

// tiles of a lattice's last layer
static int last_tiles(const nqs_ctx *c)
{
    const int w = std::min(c->L, 2 + 2 * c->K);
    return (w * w + 15) / 16;
}

// one launch: lattices of at most 24 tiles, or of more
static void inc_launch(const ConnJob *jobs, int n, hipStream_t s)
{
    if (n <= 0) return;
    BfJobs jp{};
    jp.n = n;
    size_t lds = 0;
    int64_t items = 0;
    int tiles = 0;
    for (int i = 0; i < n; ++i) {
        const nqs_ctx *c = jobs[i].c;
        BfJob &p = jp.job[i];
        p.spins = jobs[i].spins;
        p.queue = jobs[i].queue;
        p.qlen = jobs[i].qlen;
        p.capacity = jobs[i].capacity;
        p.wa = (const bf16x8 *)c->w_mfma;
        p.w1 = c->w_l1;
        p.bias = c->w_l1 + 9 * c->C;
        p.cache = (const uint16_t *)jobs[i].cache;
        p.hsum = jobs[i].hsum;
        p.dlog = jobs[i].dlog;
        p.err = c->err;
        p.L = c->L;
        p.K = c->K;
        p.P = frame_side(c);
        lds = std::max(lds, frame_bytes(c));
        tiles = std::max(tiles, last_tiles(c));
        items += jobs[i].capacity;
    }
    if (items <= 0) return;
    jp.lds = (int)lds;
    const int n_cu = jobs[0].c->n_cu;
    // one wave per configuration while its tiles fit the registers, the LDS
    // holds eight frames and there are configurations for all CUs' waves; else
    // four waves or eight (a 36x36 torus has 81 tiles).  10x10, 4 layers of 32
    // channels: one sample 62 us with one wave and 55 with four, two 63 and 57,
    // four (1600 configurations) 65 and 70
    const bool one = tiles <= 16 && 8 * lds <= kLdsMax && items >= (int64_t)4 * n_cu;
    const bool few = tiles <= 24 && items < (int64_t)4 * n_cu;
    // eight where each has a CU to itself: what chains wait for in every step is one
    // configuration's latency (20 steps of 100 chains: 12x12, 5 layers of 16, 792 ->
    // 758 us, 12x12, 8 layers, 1117 -> 1064; 357 chains of 14x14 1081 and 1079, 900
    // 1780 and 1950)
    const bool lone = few && items <= n_cu;
    if (jobs[0].c->C == 32) {
        if (one && tiles <= 9)
            launch_w<32, 1, 4, 9, 3>(jp, n_cu, items, s);
        else if (one)
            launch_w<32, 1, 4, 16, 2>(jp, n_cu, items, s);
        else if (lone)
            launch_w<32, 8, 1, 3, 2, true>(jp, n_cu, items, s);
        else if (few)
            launch_w<32, 4, 1, 6, 3, true>(jp, n_cu, items, s);
        else if (tiles <= 24)
            launch_w<32, 4, 1, 6, 3>(jp, n_cu, items, s);
        else
            launch_w<32, 8, 1, 11, 2>(jp, n_cu, items, s);
    } else {
        if (one && tiles <= 9)
            launch_w<16, 1, 4, 9, 4>(jp, n_cu, items, s);
        else if (one)
            launch_w<16, 1, 4, 16, 3>(jp, n_cu, items, s);
        else if (lone)
            launch_w<16, 8, 1, 3, 4, true>(jp, n_cu, items, s);
        else if (few)
            launch_w<16, 4, 1, 6, 4, true>(jp, n_cu, items, s);
        else if (tiles <= 24)
            launch_w<16, 4, 1, 6, 4>(jp, n_cu, items, s);
        else
            launch_w<16, 8, 1, 11, 2>(jp, n_cu, items, s);
    }
}

void mfma_inc_forward_jobs(const ConnJob *jobs, int n, hipStream_t s)
{
    // lattices of more than 24 tiles by a launch of their own: their eight waves
    // would sum the others' terms in another order than their single calls
    ConnJob part[2][kMaxConnJobs];
    int m[2] = {0, 0};
    for (int i = 0; i < n; ++i) {
        const int big = last_tiles(jobs[i].c) > 24;
        part[big][m[big]++] = jobs[i];
    }
    for (int b = 0; b < 2; ++b) inc_launch(part[b], m[b], s);
}

}  // namespace nqs

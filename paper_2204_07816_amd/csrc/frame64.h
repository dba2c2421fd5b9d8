// frame64.h -- the FP64 networks (ln cosh CNN, CNN1, CNN2) and the FP32 ln cosh
// CNN evaluated whole in LDS: one workgroup takes a configuration through every layer on a frame
// of P x P sites and C channels, so no activation of an exchanged
// configuration [Sec. 5.4.1] touches HBM.
//
// The layered form (k_conv_f64mma.hip) writes and re-reads a plane per layer;
// its matrix cores wait on A operands gathered from memory, 16 cache lines
// per load, and each layer ends in the tail of a launch.  Here the frame is
// kept as C / 2 planes of 16-byte channel pairs (FP32: C / 4 of quads), an odd number of chunks
// apart, so the 16 sites of an operand fetch are 256 contiguous bytes of LDS
// (no bank conflicts) and the two chunks of a lane sit at constant offsets.
//
// Frame: where the lattice is at most 2 F + 2 wide, F the layers' reach, it
// is the whole torus (P = L, neighbours wrap); else the exchanged pair's box
// widened by F (P = 2 F + 2, which never reaches its own edge).  Layer l is
// formed on R_l, the box widened by l sites (clamped to the torus): elsewhere
// it equals the sample's, whose activations (kept by the base pass) fill the
// ring R_{l+2} \ R_l that the next layer reads.  With `regions` off, R_l is
// the whole torus and no cache is read: the full recomputation.
//
// Layers run in place.  A wave owns 16 output columns (CNN1: both column
// blocks) and every G-th tile of 16 sites; it forms all its tiles of a layer
// at once, so one fetch of the weights serves up to NMAX tiles and the MFMAs
// of different tiles are independent.  The sums wait in registers until every
// wave has read the frame, and are then stored; ln cosh is applied to the
// accumulators meanwhile.  Operand layout, packed taps and MFMA order are
// k_conv_mma's (FP32: the vector kernels' order), so every neuron equals the
// layered form's bit for bit.
#pragma once

#include <algorithm>
#include <type_traits>

#include "nqs_internal.h"

namespace nqs {
namespace frame {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// Element type of the frame: 16-byte chunks of VEC channels of a site, the
// accumulators of v_mfma_*_16x16x4 (element i of lane group kq is row row(kq,
// i)), and the order of the channels.  FP64: K-step s of a 16-channel block is
// channels 4 kq + s, a lane's four in two chunks of natural order.  FP32:
// K-step s is channels 4 s + kq, so that the chain runs over the channels in
// ascending order: v_mfma_f32_16x16x4f32 adds its four products one by one
// with a fused multiply-add each (checked against fmaf chains on random
// operands), which makes every neuron equal the vector kernels' bit for bit;
// a lane's four sit in one chunk, channel c of a block in chunk c % 4, place c / 4.
template <typename T> struct Prec;
template <> struct Prec<double> {
    static constexpr int VEC = 2, KQ = 1;
    typedef double2 Chunk;
    typedef double4_t Acc;
    static __device__ inline int row(int kq, int i) { return kq + 4 * i; }
    static __device__ inline int plane(int ch) { return ch >> 1; }
    static __device__ inline int place(int ch) { return (ch & 1) * 8; }
    static constexpr int LANE_CH = 4, STEP_CH = 1;       // channel = LANE_CH kq + STEP_CH s
    static __device__ inline Acc mfma(double a, double b, Acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};
template <> struct Prec<float> {
    static constexpr int VEC = 4, KQ = 0;
    typedef float4 Chunk;
    typedef float4_t Acc;
    static __device__ inline int row(int kq, int i) { return 4 * kq + i; }
    static __device__ inline int plane(int ch) { return (ch >> 4) * 4 + (ch & 3); }
    static __device__ inline int place(int ch) { return ((ch >> 2) & 3) * 4; }
    static constexpr int LANE_CH = 1, STEP_CH = 4;
    static __device__ inline Acc mfma(float a, float b, Acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};

constexpr int kXcd = 8;
// CNN1's packed taps (16 channels): convolution, transposed convolution,
// block 1 (transposed convolution only) and blocks 2..
constexpr int kC1Conv = 9 * 16 * 32, kC1ConvT = 9 * 16 * 16;
constexpr int kC1First = kC1ConvT + 16, kC1Block = kC1Conv + 32 + kC1ConvT + 16;

struct FrameArgs {
    const int8_t *spins;        // [B][N]
    const uint32_t *queue;      // exchanged configurations, or
    const int64_t *offsets;     // [B + 1] queue offsets of the samples (null: one item per sample)
    int64_t cap;
    const void *w;              // packed taps of the network (double or float)
    const void *w1;             // first layer: [9][C], bias (ln cosh); canonical W [32][9], a[32]
                                // (CNN1); E [3][C] (CNN2)
    const double *wf;           // CNN2: F [C][9], b
    void *cache;                // [slots][cB][N][C] of samples b0 .., in the frame's chunks
    double *site;               // [B][N] per-site terms of the samples
    int32_t *neg;               // [B][N] negative output neurons per site (block networks)
    double *f;                  // base pass: [B] log-amplitude
    int8_t *sgn;                // base pass: [B] network sign
    int64_t cB, b0, nb;         // cache slot stride; samples of this launch
    double *dlog;               // [cap]
    int8_t *isign;              // [cap] sign ratios (block networks)
    int32_t *err;
    int L, K, P, F, regions;
    int lds;                    // LDS bytes of one configuration
    // Metropolis chains: the samples' spins are advanced n_steps steps
    int8_t *chains;             // [B][N]
    const uint32_t *rnd;        // [n_steps][B]
    const double *un;           // [n_steps][B]
    int32_t *accepted;          // [B], added to (may be null)
    int64_t B;
    int n_steps, j1, j2;
};

// what a launch does: exchanged configurations of the queue, the base pass of
// samples, or Metropolis chains
constexpr int kItems = 0, kBase = 1, kChains = 2;

__device__ inline int wrap1(int a, int P) { return a < 0 ? a + P : (a >= P ? a - P : a); }

// bytes of one channel-pair plane: an odd number of 16-byte chunks
__host__ __device__ inline int plane_bytes16(int P) { return ((P * P) | 1) * 16; }

// log of the product of v[0..n) from the product of the mantissas (in
// [1/2, 1), n <= 32: no underflow) and the sum of the exponents: one
// logarithm for n factors, to n roundings of relative size 2^-53
struct LogProd {
    double m = 1.0;
    int e = 0;
    __device__ inline void mul(double v)
    {
        m *= __builtin_amdgcn_frexp_mant(fabs(v));
        e += __builtin_amdgcn_frexp_exp(v);
    }
    __device__ inline double log() const
    {
        return fma((double)e, 0.69314718055994530942, ::log(m));
    }
};

// One lane's site of a tile: byte offset in the lane group's first channel-pair
// plane, byte steps to its four neighbours (the wraps of a torus frame are in
// them), and where its results go.
struct TileSite {
    int org, up, dn, lf, rt, to;
};

constexpr int kQuarters = 1;         // room for quarter tiles (FP64)
constexpr int kMaxSites = 1280;      // of a frame (eight waves of ten tiles)

// Accumulators of N tiles of 16 sites (NH column blocks each), of which the
// last is formed only when `last`, and of nq <= kQuarters quarter tiles of 4
// sites: bias, then the sum over the taps and input channels.  A quarter tile
// is v_mfma_f64_4x4x4f64 with its four blocks on the same 4 sites: row kq,
// column m16, the weights' operand as for a full tile and a quarter of the
// time, so a region of 36 or 100 sites is not padded to 48 or 112.
// wp: this lane's first weight.  Each K-block's weights are fetched while the
// previous block's MFMAs issue, and each tile's A operands while the previous
// tile's do.
template <typename T, int N, int CIN, int COUT, int NH>
__device__ __forceinline__ void conv_tiles(const unsigned char *fr, int SB, bool last, int nq,
                                           const TileSite (&st)[N], const TileSite (&sq)[kQuarters],
                                           const T *wp, const T *bias,
                                           typename Prec<T>::Acc (&acc)[N][NH], T (&accq)[kQuarters][NH])
{
    using Pr = Prec<T>;
    using Chunk = typename Pr::Chunk;
    constexpr int WS = Pr::STEP_CH * COUT;       // weights of successive K-steps
    constexpr int NCB = CIN / 16;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const T b = bias[16 * h];
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j][h] = (typename Pr::Acc){b, b, b, b};
#pragma unroll
        for (int q = 0; q < kQuarters; ++q) accq[q][h] = b;
    }
    T bv[4][NH];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int h = 0; h < NH; ++h) bv[s][h] = wp[s * WS + 16 * h];
#pragma unroll 1
    for (int ty = 0; ty < 3; ++ty) {
        auto row_of = [&](const TileSite &t) { return t.org + (ty == 0 ? t.up : (ty == 2 ? t.dn : 0)); };
        int row[N], rowq[kQuarters];
#pragma unroll
        for (int j = 0; j < N; ++j) row[j] = row_of(st[j]);
#pragma unroll
        for (int q = 0; q < kQuarters; ++q) rowq[q] = row_of(sq[q]);
#pragma unroll
        for (int tx = 0; tx < 3; ++tx)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                // (the last block fetches block 0's again, unused)
                const T *wn = wp + (tx * NCB + cb + 1) * 16 * COUT;
                if (tx == 2 && cb == NCB - 1 && ty == 2) wn = wp;
                T bn[4][NH];
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int h = 0; h < NH; ++h) bn[s][h] = wn[s * WS + 16 * h];
                // this lane's four channels of a site's K-block
                auto read = [&](int rw, const TileSite &t, Chunk &u, Chunk &v) {
                    const unsigned char *p = fr + (rw + (tx == 0 ? t.lf : (tx == 2 ? t.rt : 0)));
                    u = *(const Chunk *)(p + cb * (16 / Pr::VEC) * SB);
                    if constexpr (Pr::VEC == 2) v = *(const Chunk *)(p + (cb * 8 + 1) * SB);
                };
                auto unpack = [](const Chunk &u, const Chunk &v, T (&av)[4]) {
                    av[0] = u.x;
                    av[1] = u.y;
                    if constexpr (Pr::VEC == 2) {
                        av[2] = v.x;
                        av[3] = v.y;
                    } else {
                        av[2] = u.z;
                        av[3] = u.w;
                    }
                };
                Chunk u, v;
                read(row[0], st[0], u, v);
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    Chunk un = u, vn = v;
                    if (j + 1 < N) read(row[j + 1], st[j + 1], un, vn);
                    T av[4];
                    unpack(u, v, av);
                    if (j + 1 < N || last)
#pragma unroll
                        for (int s = 0; s < 4; ++s)
#pragma unroll
                            for (int h = 0; h < NH; ++h)
                                acc[j][h] = Pr::mfma(av[s], bv[s][h], acc[j][h]);
                    u = un;
                    v = vn;
                }
                if constexpr (Pr::KQ > 0) {
#pragma unroll
                    for (int q = 0; q < kQuarters; ++q)
                        if (q < nq) {
                            read(rowq[q], sq[q], u, v);
                            T av[4];
                            unpack(u, v, av);
#pragma unroll
                            for (int s = 0; s < 4; ++s)
#pragma unroll
                                for (int h = 0; h < NH; ++h)
                                    accq[q][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                        av[s], bv[s][h], accq[q][h], 0, 0, 0);
                        }
                }
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int h = 0; h < NH; ++h) bv[s][h] = bn[s][h];
            }
        wp += 3 * NCB * 16 * COUT;
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

// R_l in frame coordinates: start and extent in x and y
struct Region {
    int x0, y0, w, h;
};

// W waves form a configuration.  PK > 1 (W = 1 only): the workgroup holds PK
// such waves, each with its own frame and items and no barrier between them; a
// workgroup of four puts one on every SIMD, where single-wave workgroups would
// fill the SIMDs unevenly (11 of 10x10 fit a CU).
//
// Chains: a chain stays with its workgroup for all its steps; its spins and
// the per-site terms of its configuration live in LDS.  Each proposal whose
// two spins differ is evaluated in full (the layers in between are not kept),
// accepted when u < exp(2 dlog), and the terms then replace the chain's.
template <typename T, int C, int NET, int W, int PK, int NMAX, int MODE, int EU>
__global__ void __launch_bounds__(W * PK * 64, EU)
k_frame64(FrameArgs a)
{
    static_assert(PK == 1 || W == 1, "only single waves share a workgroup");
    constexpr bool BASE = MODE == kBase, CHAIN = MODE == kChains;
    constexpr int NT = W * 64;
    auto sync = [] {
        if constexpr (W == 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };
    using Pr = Prec<T>;
    using Chunk = typename Pr::Chunk;
    constexpr int CHK = C / Pr::VEC;                 // 16-byte chunks per site
    constexpr int NHB = NET == kNetCnn1 ? 1 : C / 16;   // waves per tile (one column block each)
    constexpr int G = W / NHB;                       // tile groups
    static_assert(G >= 1 && G * NHB == W, "waves split into column blocks and tile groups");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    // sums of the output terms of 64 sites (CNN2: 16), in the order of the sites:
    // the same parts and the same order whatever W is, which depends on the number
    // of items for 16 channels (ONE: it does not, and a wave's terms are one part)
    constexpr bool ONE = C == 32 && NET != kNetCnn2;
    __shared__ double red[W == 1 ? 1 : (NET == kNetCnn2 ? kMaxSites / 16 : kMaxSites / 64)];
    __shared__ int nred[W];
    const int pk = PK > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    unsigned char *fr = lds + pk * a.lds;
    const int tid = PK > 1 ? threadIdx.x & 63 : threadIdx.x, lane = tid & 63;
    const int wave = PK > 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m16 = lane & 15, kq = lane >> 4;
    const int hb = wave % NHB, grp = wave / NHB;
    const int L = a.L, N = L * L, P = a.P, F = a.F, K = a.K;
    const bool torus = MODE != kItems || P == L;
    const int SB = plane_bytes16(P);
    int8_t *sf = (int8_t *)(fr + CHK * SB);          // exchanged spins around R_1
    // CNN2, 32 channels: z of the column blocks' first columns; F as [9][C], b
    double *zb = (double *)(fr + CHK * SB + (((P + 2) * (P + 2) + 15) & ~15));
    double *fw = zb + (NET == kNetCnn2 && C == 32 ? 2 * P * P : 0);
    // chains: per-site terms of the chain's and the proposed configuration, spins
    double *hs = fw + (NET == kNetCnn2 ? 9 * C + 1 : 0), *hn = hs + N;
    int8_t *cs = (int8_t *)(hn + N);
    const int S = NET == kNetLnCosh ? K : 2 * K;     // layers stored in the frame
    const int ncache = NET == kNetCnn2 ? S : S - 1;  // of them kept by the base pass
    if constexpr (NET == kNetCnn2) {
        for (int q = tid; q < 9 * C; q += NT) fw[(q % 9) * C + q / 9] = a.wf[q];
        if (tid == 0) fw[9 * C] = a.wf[9 * C];
        sync();
    }

    int64_t u, u_end, u_step;
    if constexpr (MODE != kItems) {
        u = (int64_t)blockIdx.x * PK + pk;
        u_end = a.nb;
        u_step = (int64_t)gridDim.x * PK;
    } else {
        // the launch's items, split into XCD-contiguous ranges (the grid is a
        // multiple of 8), so that items of one sample share an L2
        const int64_t q0 = a.offsets ? a.offsets[a.b0] : a.b0;
        const int64_t q1 = a.offsets ? a.offsets[a.b0 + a.nb] : a.b0 + a.nb;
        const int64_t lim = min(q1, a.cap), seg = (lim - q0 + kXcd - 1) / kXcd;
        const int xcd = blockIdx.x % kXcd;
        u = q0 + xcd * seg + blockIdx.x / kXcd * PK + pk;
        u_end = min(lim, q0 + (xcd + 1) * seg);
        u_step = gridDim.x / kXcd * PK;
    }
    // a chain: step -1 evaluates its configuration, then its proposals follow
    int step = -1, n_acc = 0;
    uint32_t rnd = 0;
    double un = 0.0, un_next = 0.0;
    for (; u < u_end;) {
        int s, qi = -1, qj = -1, ax = 0, ay = 0, w0 = 2, h0 = 2;
        if constexpr (MODE != kItems) {
            s = (int)(a.b0 + u);
            if constexpr (CHAIN) {
                auto numbers = [&](int t) {
                    if (t < a.n_steps) {
                        rnd = a.rnd[(int64_t)t * a.B + s];
                        un_next = a.un[(int64_t)t * a.B + s];
                    }
                };
                if (step < 0) {
                    for (int p = tid; p < N; p += NT) {
                        cs[p] = a.chains[(int64_t)s * N + p];
                        hs[p] = 0.0;
                    }
                    n_acc = 0;
                    numbers(0);
                    sync();
                } else if (step == a.n_steps) {
                    for (int p = tid; p < N; p += NT) a.chains[(int64_t)s * N + p] = cs[p];
                    if (tid == 0 && a.accepted) a.accepted[s] += n_acc;
                    step = -1;
                    u += u_step;
                    sync();
                    continue;
                } else {
                    const int b = proposal_bond(rnd, N, a.j1, a.j2), tau = b & 3;
                    qi = b >> 2;
                    const int xi = qi % L, yi = qi / L;
                    qj = wrap1(yi + bond_dy(tau), L) * L + wrap1(xi + bond_dx(tau), L);
                    un = un_next;
                    numbers(step + 1);
                    // equal spins: S' = S, never accepted
                    if (__builtin_amdgcn_readfirstlane(cs[qi] == cs[qj])) {
                        ++step;
                        continue;
                    }
                }
            }
        } else {
            const uint32_t e = a.queue[u];
            const int b = item_bond(e), tau = b & 3, i0 = b >> 2;
            const int xi = i0 % L, yi = i0 / L;
            s = item_sample(e);
            qi = i0;
            qj = wrap1(yi + bond_dy(tau), L) * L + wrap1(xi + bond_dx(tau), L);
            ax = xi;
            ay = (tau == 3) ? wrap1(yi - 1, L) : yi;
            w0 = (tau == 1) ? 1 : 2;
            h0 = (tau == 0) ? 1 : 2;
        }
        const bool part = MODE == kItems && a.regions;
        auto region = [&](int l) {
            Region r{0, 0, L, L};
            if (part) {
                if (w0 + 2 * l < L) r.x0 = torus ? wrap1(ax - l, L) : F - l, r.w = w0 + 2 * l;
                if (h0 + 2 * l < L) r.y0 = torus ? wrap1(ay - l, L) : F - l, r.h = h0 + 2 * l;
            }
            return r;
        };
        // lattice site of frame position (fx, fy); a torus frame is the lattice
        auto site_of = [&](int fx, int fy) {
            if (torus) return fy * L + fx;
            int x = ax - F + fx, y = ay - F + fy;
            x += x < 0 ? L : (x >= L ? -L : 0);
            y += y < 0 ? L : (y >= L ? -L : 0);
            return y * L + x;
        };
        auto inside = [&](int f) { return f >= P ? f - P : f; };
        // the exchanged configuration on R_1 and one site around it, row by row
        // (the wraps of the torus are in the array, so the first layer's
        // neighbours are at constant steps)
        const Region r1 = region(1);
        const int sw = r1.w + 2, sn = sw * (r1.h + 2);
        const uint32_t smul = ((1u << 20) + sw - 1) / sw;
        auto halo = [&](int e, int &fx, int &fy) {
            const int v = (int)(((uint32_t)e * smul) >> 20);
            fx = wrap1(r1.x0 + e - v * sw - 1, P);
            fy = wrap1(r1.y0 + v - 1, P);
        };
        for (int e = tid; e < sn; e += NT) {
            int fx, fy;
            halo(e, fx, fy);
            int q = site_of(fx, fy);
            q = (q == qi) ? qj : ((q == qj) ? qi : q);
            sf[e] = CHAIN ? cs[q] : a.spins[(int64_t)s * N + q];
        }
        sync();
        const T *w1 = (const T *)a.w1;
        // first layer from the spins: CNN2's embedding (R_2: the whole array)
        if constexpr (NET == kNetCnn2) {
            const int co = tid % C;
            for (int e = tid / C; e < sn; e += NT / C) {
                int fx, fy;
                halo(e, fx, fy);
                const int8_t sv = sf[e];
                *(T *)(fr + Pr::plane(co) * SB + (fy * P + fx) * 16 + Pr::place(co)) =
                    w1[(sv == 0 ? 0 : (sv > 0 ? 1 : 2)) * C + co];
            }
        } else {
            // ln cosh (bias, then the taps), or CNN1's convolution and
            // channel-pair max, on R_1
            const uint32_t mul = ((1u << 20) + r1.w - 1) / r1.w;
            const int co = tid % C;
            T wz0[9], wz1[9], b0, b1 = 0;
            if constexpr (NET == kNetLnCosh) {
#pragma unroll
                for (int t = 0; t < 9; ++t) wz0[t] = w1[t * C + co];
                b0 = w1[9 * C + co];
            } else {
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    wz0[t] = w1[(2 * co) * 9 + t];
                    wz1[t] = w1[(2 * co + 1) * 9 + t];
                }
                b0 = w1[18 * C + 2 * co];
                b1 = w1[18 * C + 2 * co + 1];
            }
            unsigned char *frc = fr + Pr::plane(co) * SB + Pr::place(co);
            for (int p = tid / C; p < r1.w * r1.h; p += NT / C) {
                const int v = (int)(((uint32_t)p * mul) >> 20), x = p - v * r1.w;
                const int8_t *nb = sf + v * sw + x;
                T z0 = b0, z1 = b1;
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const T sv = (T)nb[t / 3 * sw + t % 3];
                    z0 = fma(wz0[t], sv, z0);
                    if constexpr (NET == kNetCnn1) z1 = fma(wz1[t], sv, z1);
                }
                *(T *)(frc + (inside(r1.y0 + v) * P + inside(r1.x0 + x)) * 16) =
                    NET == kNetCnn1 ? ((z1 > z0) ? z1 : z0) : ln_cosh_fwd(z0);
            }
        }
        // ring R_{l+2} \ R_l from the sample's activations of layer l: the
        // threads span a stretch of a row (site, channel pair), the rows are
        // taken four at a time; a row's offsets are scalar
        auto ring = [&](int l) {
            constexpr int XP = NT / CHK;             // sites per stretch
            const Region in = region(l), out = region(l + 2);
            if (in.w == out.w && in.h == out.h) return;
            const T *src = (const T *)a.cache + ((int64_t)(l - 1) * a.cB + (s - a.b0)) * N * C;
            const int c = tid % CHK;
            for (int xb = 0; xb < out.w; xb += XP) {
                const int x = xb + tid / CHK;
                const int fx = inside(out.x0 + min(x, out.w - 1));
                const int dx = fx - in.x0 + (fx < in.x0 ? P : 0);
                const bool side = x < out.w && dx >= in.w, live = x < out.w;
                const int lx = torus ? fx : wrap1(ax - F + fx, L);
                const T *gx = src + lx * C + Pr::VEC * c;
                unsigned char *fc = fr + c * SB + fx * 16;
                // row v of the stretch: frame row, and whether this lane copies
                auto row = [&](int v, bool &on) {
                    const int fy = inside(out.y0 + min(v, out.h - 1));
                    const int dy = fy - in.y0 + (fy < in.y0 ? P : 0);
                    on = v < out.h && (dy >= in.h ? live : side);
                    return fy;
                };
                auto get = [&](int fy, bool on) {
                    const int ly = torus ? fy : wrap1(ay - F + fy, L);
                    return *(const Chunk *)(gx + (on ? ly * L * C : 0));
                };
                for (int v = 0; v < out.h; v += 4) {
                    bool o0, o1, o2, o3;
                    const int f0 = row(v, o0), f1 = row(v + 1, o1), f2 = row(v + 2, o2), f3 = row(v + 3, o3);
                    if (__ballot(o0 || o1 || o2 || o3) == 0) continue;
                    const Chunk d0 = get(f0, o0), d1 = get(f1, o1), d2 = get(f2, o2), d3 = get(f3, o3);
                    if (o0) *(Chunk *)(fc + f0 * P * 16) = d0;
                    if (o1) *(Chunk *)(fc + f1 * P * 16) = d1;
                    if (o2) *(Chunk *)(fc + f2 * P * 16) = d2;
                    if (o3) *(Chunk *)(fc + f3 * P * 16) = d3;
                }
            }
        };
        // base pass: the frame (the whole torus) becomes cache slot l - 1
        auto keep = [&](int l) {
            T *dst = (T *)a.cache + ((int64_t)(l - 1) * a.cB + (s - a.b0)) * N * C;
            for (int q = tid; q < N * CHK; q += NT)
                *(Chunk *)(dst + Pr::VEC * q) = *(const Chunk *)(fr + (q % CHK) * SB + (q / CHK) * 16);
        };
        if constexpr (NET != kNetCnn2)
            if (part && S > 1) ring(1);
        sync();

        for (int l = NET == kNetCnn2 ? 1 : 2; l <= S; ++l) {
            if constexpr (BASE)
                if (a.cache && l - 1 >= 1) keep(l - 1);
            const bool pairs = NET == kNetCnn1 && (l & 1);   // CNN1 convolution 16 -> 32
            const T *wl, *bias;
            if constexpr (NET == kNetLnCosh) {
                wl = (const T *)a.w + (int64_t)(l - 2) * (9 * C * C + C);
                bias = wl + 9 * C * C;
            } else if constexpr (NET == kNetCnn1) {
                const int k = (l - 1) >> 1;
                wl = k == 0 ? (const T *)a.w : (const T *)a.w + kC1First + (int64_t)(k - 1) * kC1Block;
                if (k > 0 && !pairs) wl += kC1Conv + 32;
                bias = wl + (pairs ? kC1Conv : kC1ConvT);
            } else {
                wl = (const T *)a.w + (int64_t)((l - 1) >> 1) * (36 * C * C + 2 * C) + ((l & 1) ? 0 : 9 * C * C + C);
                bias = wl + 9 * C * C;
            }
            const Region r = region(l);
            const int nl = r.w * r.h;
            const uint32_t mul = ((1u << 20) + r.w - 1) / r.w;
            // tiles grp + G j of this wave; the workgroup's largest count is
            // the compiled one, and a wave with one less skips the last; the
            // sites past the full tiles are quarter tiles of the first group
            // with fewer tiles, or a full tile if there are more than 8
            int TF = nl >> 4, NQ = ((nl & 15) + 3) >> 2;
            if (TF == 0 || NQ > Pr::KQ) ++TF, NQ = 0;
            const int nq = grp == TF % G ? NQ : 0;
            auto site = [&](int q) {
                TileSite t;
                const int p = min(q, nl - 1);
                const int v = (int)(((uint32_t)p * mul) >> 20);
                const int fx = inside(r.x0 + p - v * r.w), fy = inside(r.y0 + v);
                const int f = fy * P + fx;
                t.org = f * 16 + (Pr::VEC == 2 ? 2 : 1) * kq * SB;
                t.to = (q < nl ? f : P * P) * 16;   // past the end: the planes' spare chunk
                t.up = (fy == 0 ? P - 1 : -1) * P * 16;
                t.dn = (fy == P - 1 ? 1 - P : 1) * P * 16;
                t.lf = (fx == 0 ? P - 1 : -1) * 16;
                t.rt = (fx == P - 1 ? 1 - P : 1) * 16;
                return t;
            };
            auto layer = [&](auto count, auto nhc) {
                constexpr int TN = decltype(count)::value, NH = decltype(nhc)::value;
                const bool last = grp + G * (TN - 1) < TF;
                TileSite st[TN], sq[kQuarters];
#pragma unroll
                for (int j = 0; j < TN; ++j) st[j] = site((grp + G * j) * 16 + m16);
#pragma unroll
                for (int q = 0; q < kQuarters; ++q) sq[q] = site(TF * 16 + 4 * q + (lane & 3));
                typename Pr::Acc acc[TN][NH];
                T accq[kQuarters][NH];
                conv_tiles<T, TN, C, C * NH, NH>(fr, SB, last, nq, st, sq,
                                              wl + Pr::LANE_CH * kq * C * NH + 16 * hb + m16,
                                              bias + 16 * hb + m16, acc, accq);
                const bool c2max = NET == kNetCnn2 && (l & 1);
                if constexpr (NET == kNetLnCosh) {
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[j][0][i] = ln_cosh_fwd(acc[j][0][i]);
#pragma unroll
                    for (int q = 0; q < kQuarters; ++q)
                        if (q < nq) accq[q][0] = ln_cosh_fwd(accq[q][0]);
                }
                if constexpr (NET == kNetCnn2 && C == 32) {
                    // the neighbouring column block's waves need column 0's z
                    auto lend = [&](int p, double z) {
                        if (p < nl) zb[hb * P * P + p] = z;
                    };
                    if (c2max && m16 == 0) {
#pragma unroll
                        for (int j = 0; j < TN; ++j)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (j + 1 < TN || last) lend((grp + G * j) * 16 + kq + 4 * i, acc[j][0][i]);
#pragma unroll
                        for (int q = 0; q < kQuarters; ++q)
                            if (q < nq) lend(TF * 16 + 4 * q + kq, accq[q][0]);
                    }
                }
                sync();                      // every read of the frame for layer l is done
                const int ch = 16 * hb + m16;
                unsigned char *frc = fr + Pr::plane(ch) * SB + Pr::place(ch);
                // one result of this lane's column: position p, row `row` of a tile
                auto store = [&](int p, int to, int row, const T (&zs)[NH]) {
                    T z = zs[0];
                    if constexpr (NH == 2) {
                        z = (zs[1] > z) ? zs[1] : z;
                    } else if constexpr (NET == kNetCnn2) {
                        if (c2max) {
                            double z1 = __shfl(z, (lane & 48) | ((m16 + 1) & 15), 64);
                            if constexpr (C == 32)
                                if (m16 == 15 && p < nl) z1 = zb[(1 - hb) * P * P + p];
                            z = (z1 > z) ? z1 : z;
                        }
                    }
                    *(T *)(frc + __shfl(to, row, 64)) = z;
                };
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (j + 1 < TN || last)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            T zs[NH];
#pragma unroll
                            for (int h = 0; h < NH; ++h) zs[h] = acc[j][h][i];
                            store((grp + G * j) * 16 + Pr::row(kq, i), st[j].to, Pr::row(kq, i), zs);
                        }
#pragma unroll
                for (int q = 0; q < kQuarters; ++q)
                    if (q < nq) store(TF * 16 + 4 * q + kq, sq[q].to, kq, accq[q]);
            };
            const int n = (TF + G - 1) / G;
            if (pairs)
                with_count<NMAX>(n, [&](auto t) { layer(t, std::integral_constant<int, NET == kNetCnn1 ? 2 : 1>{}); });
            else
                with_count<NMAX>(n, [&](auto t) { layer(t, std::integral_constant<int, 1>{}); });
            if (part && l <= ncache) ring(l);
            sync();
        }

        // the output neurons: per-site terms, against the sample's
        double total = 0.0;
        int dn = 0, parts = 0;
        auto take = [&](int site, double v, int neg) {
            const int64_t o = (int64_t)s * N + site;
            if constexpr (BASE) {
                a.site[o] = v;
                if constexpr (NET != kNetLnCosh) a.neg[o] = neg, dn += neg;
                return v;
            } else if constexpr (CHAIN) {
                hn[site] = v;
                return v - hs[site];
            } else {
                if constexpr (NET != kNetLnCosh) dn += neg - a.neg[o];
                return v - a.site[o];
            }
        };
        // parts i ..: the lanes' terms t in a fixed tree (lanes apart by `from` and more)
        auto part_sum = [&](int i, auto &t, auto from) {
#pragma unroll
            for (int off = 32; off >= decltype(from)::value; off >>= 1)
#pragma unroll
                for (double &x : t) x += __shfl_xor(x, off);
            for (double &x : t)
                if constexpr (W == 1)
                    total += x;
                else if (lane == 0)
                    red[i] = x;
        };
        if constexpr (NET == kNetCnn2) {
            if constexpr (BASE)
                if (a.cache) keep(S);
            // y on R_{2K+1}: four lanes per site, each every fourth channel pair
            const Region r = region(S + 1);
            const int nl = r.w * r.h;
            const uint32_t mul = ((1u << 20) + r.w - 1) / r.w;
            const int pt = tid & 3;
            parts = (nl + 15) >> 4;
            for (int p0 = wave * 16; p0 < nl; p0 += NT / 4) {
                const int p = min(p0 + (lane >> 2), nl - 1);
                const int v = (int)(((uint32_t)p * mul) >> 20);
                const int fx = inside(r.x0 + p - v * r.w), fy = inside(r.y0 + v);
                double y = 0.0;
#pragma unroll 1
                for (int t = 0; t < 9; ++t) {
                    const unsigned char *q = fr + pt * SB +
                        (wrap1(fy + t / 3 - 1, P) * P + wrap1(fx + t % 3 - 1, P)) * 16;
                    const double *wt = fw + t * C + 2 * pt;
#pragma unroll
                    for (int c = 0; c < CHK / 4; ++c) {
                        const double2 h = *(const double2 *)(q + 4 * c * SB);
                        y = fma(wt[8 * c], h.x, y);
                        y = fma(wt[8 * c + 1], h.y, y);
                    }
                }
                y += __shfl_xor(y, 1);
                y += __shfl_xor(y, 2);
                y += fw[9 * C];
                double t[1] = {0.0};
                if (pt == 0 && p0 + (lane >> 2) < nl) t[0] = take(site_of(fx, fy), log(fabs(y)), y < 0.0);
                part_sum(p0 >> 4, t, std::integral_constant<int, 4>{});
            }
        } else {
            const Region r = region(S);
            const int nl = r.w * r.h;
            const uint32_t mul = ((1u << 20) + r.w - 1) / r.w;
            // one site's term
            auto term = [&](int p) {
                const int v = (int)(((uint32_t)p * mul) >> 20);
                const int fx = inside(r.x0 + p - v * r.w), fy = inside(r.y0 + v);
                const unsigned char *q = fr + (fy * P + fx) * 16;
                if constexpr (NET == kNetLnCosh) {
                    double hs = 0.0;           // the channels in order
#pragma unroll
                    for (int c0 = 0; c0 < C; c0 += 16) {
                        Chunk h[16 / Pr::VEC];
#pragma unroll
                        for (int c = 0; c < 16 / Pr::VEC; ++c)
                            h[c] = *(const Chunk *)(q + (c0 / Pr::VEC + c) * SB);
#pragma unroll
                        for (int c = 0; c < 16; ++c) {
                            if constexpr (Pr::VEC == 2) {
                                hs += c & 1 ? h[c >> 1].y : h[c >> 1].x;
                            } else {
                                const Chunk &k = h[c & 3];
                                hs += (double)(c >> 2 == 0 ? k.x : (c >> 2 == 1 ? k.y : (c >> 2 == 2 ? k.z : k.w)));
                            }
                        }
                    }
                    return take(site_of(fx, fy), hs, 0);
                } else {
                    LogProd lp;
                    int neg = 0;
#pragma unroll
                    for (int c = 0; c < CHK; ++c) {
                        const double2 h = *(const double2 *)(q + c * SB);
                        lp.mul(h.x);
                        lp.mul(h.y);
                        neg += (h.x < 0.0) + (h.y < 0.0);
                    }
                    return take(site_of(fx, fy), lp.log(), neg);
                }
            };
            if constexpr (ONE) {
                double t[1] = {0.0};
                for (int p = tid; p < nl; p += NT) t[0] += term(p);
                part_sum(wave, t, std::integral_constant<int, 1>{});
            } else {
                parts = (nl + 63) >> 6;
                // (one wave: two parts' trees at a time)
                constexpr int PT = W == 1 ? 2 : 1;
#pragma unroll 1
                for (int p0 = wave * 64; p0 < nl; p0 += PT * NT) {
                    double t[PT];
#pragma unroll
                    for (int i = 0; i < PT; ++i)
                        t[i] = p0 + 64 * i + lane < nl ? term(p0 + 64 * i + lane) : 0.0;
                    part_sum(p0 >> 6, t, std::integral_constant<int, 1>{});
                }
            }
        }
        if constexpr (NET != kNetLnCosh) {
            for (int off = 32; off > 0; off >>= 1) dn += __shfl_xor(dn, off);
            if constexpr (W > 1)
                if (lane == 0) nred[wave] = dn;
        }
        sync();                              // the frame is free again
        auto sum_parts = [&] {               // (four loads at a time)
            double v = total;
            if constexpr (W > 1 && ONE)
                for (int i = 0; i < W; ++i) v += red[i];
            else if constexpr (W > 1)
                for (int i = 0; i < parts; i += 4) {
                    double t[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) t[j] = red[min(i + j, parts - 1)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) v += i + j < parts ? t[j] : 0.0;
                }
            return v;
        };
        if constexpr (CHAIN) {
            const double v = sum_parts();
            if (tid == 0 && !isfinite(v)) atomicOr(a.err, kErrNonFinite);
            if (__builtin_amdgcn_readfirstlane(step < 0 || un < exp(2.0 * v))) {
                for (int p = tid; p < N; p += NT) hs[p] = hn[p];
                if (step >= 0) {
                    if (tid == 0) {
                        const int8_t t = cs[qi];
                        cs[qi] = cs[qj];
                        cs[qj] = t;
                    }
                    ++n_acc;
                }
                sync();
            }
            ++step;
            continue;
        }
        if (tid == 0) {
            const double v = sum_parts();
            int ng = W > 1 ? 0 : dn;
            if constexpr (W > 1 && NET != kNetLnCosh)
                for (int w = 0; w < W; ++w) ng += nred[w];
            if (!isfinite(v)) atomicOr(a.err, kErrNonFinite);
            const int8_t sg = (ng & 1) ? -1 : 1;
            if constexpr (BASE) {
                a.f[s] = v;
                if constexpr (NET != kNetLnCosh) a.sgn[s] = sg;
            } else {
                a.dlog[u] = v;
                if constexpr (NET != kNetLnCosh) a.isign[u] = sg;
            }
        }
        u += u_step;
    }
}

// channels of the frame: a ln cosh network's, filled up to 16 or 32 with
// neurons of zero weight (their ln cosh is 0, so every sum keeps its terms)
inline int frame_ch(const nqs_ctx *c)
{
    return c->net != kNetLnCosh ? c->C : (c->C <= 16 ? 16 : 32);
}

inline size_t frame_lds(const nqs_ctx *c, int P, bool chains = false)
{
    size_t n = (size_t)(frame_ch(c) / (c->dtype == NQS_FP32 ? 4 : 2)) * plane_bytes16(P) + (size_t)(((P + 2) * (P + 2) + 15) & ~15);
    if (c->net == kNetCnn2) n += sizeof(double) * ((c->C == 32 ? 2 * (size_t)P * P : 0) + 9 * c->C + 1);
    if (chains) n += (size_t)c->N * (2 * sizeof(double) + 1);
    return (n + 15) & ~(size_t)15;
}

constexpr size_t kLdsMax = 160 * 1024 - 1024;   // (the part sums are beside the frame)

// layers' reach: the last stencil's region is the box widened by this much
inline int frame_reach(const nqs_ctx *c)
{
    return c->net == kNetLnCosh ? c->K : (c->net == kNetCnn1 ? 2 * c->K : 2 * c->K + 1);
}

// Tiles of the largest layer: the whole torus, or with `regions` the pair's box
// widened by the stored layers' reach.  FP64's last few sites go to quarter tiles.
inline int frame_tiles(const nqs_ctx *c, bool regions)
{
    const int S = c->net == kNetLnCosh ? c->K : 2 * c->K;
    const int wd = regions ? std::min(c->L, 2 + 2 * S) : c->L;
    return (wd * wd + 15 - (c->dtype == NQS_FP32 ? 0 : 4 * kQuarters)) / 16;
}

// tiles that W waves of NMAX each can form
inline int frame_room(const nqs_ctx *c, int W, int NMAX)
{
    return W / (c->net == kNetCnn1 ? 1 : frame_ch(c) / 16) * NMAX;
}

template <typename T, int C, int NET, int W, int PK, int NMAX, int MODE, int EU>
void launch_w(const nqs_ctx *c, FrameArgs a, int64_t items, hipStream_t s)
{
    const auto kernel = k_frame64<T, C, NET, W, PK, NMAX, MODE, EU>;
    if (frame_tiles(c, MODE == kItems && a.regions) > frame_room(c, W, NMAX))
        return refuse_launch("k_frame64: more tiles than the waves can form");
    a.lds = (int)frame_lds(c, a.P, MODE == kChains);
    const int lds = a.lds * PK;
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    int occ = 1;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, W * PK * 64, lds);
    int64_t grid = (int64_t)std::max(occ, 1) * std::max(c->n_cu, 1);
    grid = std::max<int64_t>(1, std::min(grid, (items + PK - 1) / PK));
    if (MODE == kItems) grid = (grid + kXcd - 1) / kXcd * kXcd;
    NQS_LAUNCH(kernel, dim3((unsigned)grid), dim3(W * PK * 64), lds, s, a);
}

// Workgroup shapes of the exchanged pass and of chains: waves per
// configuration, configurations per workgroup, tiles a wave can form at once.
// The base pass runs the last.
struct FrameShape {
    int W, PK, NMAX;
};
constexpr FrameShape kShapes16[4] = {{1, 4, 7}, {1, 4, 10}, {4, 1, 5}, {8, 1, 10}};
constexpr FrameShape kShapes32[3] = {{4, 1, 5}, {4, 1, 8}, {8, 1, 10}};

template <typename T, int C, int NET, int MODE>
void launch_m(const nqs_ctx *c, const FrameArgs &a, int64_t items, int shape, hipStream_t s)
{
    if constexpr (C == 16) {
        constexpr int EU = NET == kNetCnn1 ? 2 : 3;
        if (shape == 0) return launch_w<T, C, NET, 1, 4, 7, MODE, EU>(c, a, items, s);
        if constexpr (NET != kNetCnn1 && MODE == kItems)
            if (shape == 1) return launch_w<T, C, NET, 1, 4, 10, MODE, 2>(c, a, items, s);
        if (shape == 2) return launch_w<T, C, NET, 4, 1, 5, MODE, EU>(c, a, items, s);
    } else {
        if (shape == 0) return launch_w<T, C, NET, 4, 1, 5, MODE, 3>(c, a, items, s);
        if constexpr (MODE == kItems)
            if (shape == 1) return launch_w<T, C, NET, 4, 1, 8, MODE, 2>(c, a, items, s);
    }
    launch_w<T, C, NET, 8, 1, 10, MODE, 2>(c, a, items, s);
}

template <typename T, int C, int NET>
void launch_c(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape,
              hipStream_t s)
{
    if (mode == kBase)
        launch_w<T, C, NET, 8, 1, 10, kBase, 2>(c, a, items, s);
    else if (mode == kChains)
        launch_m<T, C, NET, kChains>(c, a, items, shape, s);
    else
        launch_m<T, C, NET, kItems>(c, a, items, shape, s);
}

// one translation unit per network (k_frame64_*.hip)
void launch_ln16(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s);
void launch_ln32(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s);
void launch_ln16f(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s);
void launch_ln32f(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s);
void launch_cnn1(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s);
void launch_cnn2_16(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s);
void launch_cnn2_32(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s);

}  // namespace frame
}  // namespace nqs

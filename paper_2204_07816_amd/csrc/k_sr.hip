// k_sr.hip -- stochastic reconfiguration [Sec. 3.2: SR gradients and
// covariance give the parameter update delta; Sec. 5.4.1 "Distributed SR
// computation"].  The paper forms the [R, R] covariance and factorises it;
// here the same system
//     (S + lambda I) x = F,  S = Obar^T Obar / Ns,  F = Obar^T (E - Ebar) / Ns,
// Obar = O - mean(O), is solved by conjugate gradient with S applied
// matrix-free as two streaming passes over O per iteration (HBM bound).
// O is read as FP32 or FP64; every product, sum and dot is FP64.  Scalars
// (alpha, beta, r.r) stay on the device, so the solve never synchronises
// with the host and can be captured in a graph.  All reductions are two-stage
// with a fixed order (deterministic), the same for every launch shape.  One
// iteration is five launches (p, from the second one on; Obar p; the partial
// column sums of Obar^T u; Ap with p.Ap; the update of x and r), three where P is
// small (k_ap_small is p, the column sums and Ap in one); each finishes the
// previous one's reduction itself (see k_rowdot).
#include <algorithm>

#include "nqs_internal.h"

namespace nqs {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxChunks = 64;

// No launch writes a flag that it reads: the waves of a block have to agree on
// it before their barriers.  done[it & 1] is written by the first launch of
// iteration it (k_dot_final for it = 0) and read by the others of that
// iteration; stop is written by the last and read by the first of the next.
struct SrCtl {
    double rr, ff, alpha, beta, mean, var;
    double rrv[2];   // r.r at the start of iteration it, in slot it & 1
    int done[2];     // no work left in iteration it, in slot it & 1
    int stop;        // p.Ap <= 0: nothing after that iteration
    int it;
};

__device__ inline double ld(const float *p, int64_t i) { return (double)p[i]; }
__device__ inline double ld(const double *p, int64_t i) { return p[i]; }

// Sum over the block's kThreads values, the binary tree of offsets 128 .. 1, in
// every thread.  One barrier, and every wave sums for itself.
__device__ __forceinline__ double tree_sum(const double *sh)
{
    static_assert(kThreads == 256, "four waves");
    const int l = threadIdx.x & 63;
    double v = (sh[l] + sh[l + 128]) + (sh[l + 64] + sh[l + 192]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return __shfl(v, 0, 64);
}

// sh: kThreads values, used by no call before the next barrier
__device__ __forceinline__ double block_sum(double v, double *sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    return tree_sum(sh);
}

// 16-byte vectors of O: VW consecutive elements (4 FP32 or 2 FP64)
template <typename OT, int VW> struct Vec;
template <> struct Vec<float, 4> {
    typedef float4 T;
    static __device__ inline void get(const float *q, double (&o)[4])
    {
        const float4 v = *reinterpret_cast<const float4 *>(q);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
};
template <> struct Vec<double, 2> {
    static __device__ inline void get(const double *q, double (&o)[2])
    {
        const double2 v = *reinterpret_cast<const double2 *>(q);
        o[0] = v.x; o[1] = v.y;
    }
};
template <typename OT> struct Vec<OT, 1> {
    static __device__ inline void get(const OT *q, double (&o)[1]) { o[0] = (double)q[0]; }
};

// part[c][p] = sum_{s in chunk c} (O[s][p] - sub[p]) * wt[s]   (sub / wt may be null)
// A wave owns 64 VW consecutive columns of one chunk (VW elements a lane, 16
// bytes where that leaves waves for the whole chip) and keeps 16 rows of loads
// in flight; every column sums its rows in order whatever VW is.  In blocks of
// four waves, a load or two in flight, 512 rows of 28,064 floats took 21 us, now
// 9.7; 2048 rows of 46,560 are bound by HBM, 64 us before and now (6 TB/s).
template <typename OT, int VW>
__global__ void __launch_bounds__(64)
k_colsum(const OT *__restrict__ O, int64_t B, int64_t P, const double *__restrict__ sub,
         const double *__restrict__ wt, int64_t rows_per_chunk, double *__restrict__ part,
         const int *done)
{
    if (done && *done) return;
    const int64_t p = ((int64_t)blockIdx.x * 64 + threadIdx.x) * VW;
    if (p >= P) return;
    const int64_t s0 = (int64_t)blockIdx.y * rows_per_chunk;
    const int64_t s1 = min(B, s0 + rows_per_chunk);
    double m[VW], acc[VW];
#pragma unroll
    for (int q = 0; q < VW; ++q) {
        m[q] = sub ? sub[p + q] : 0.0;
        acc[q] = 0.0;
    }
#pragma unroll 16
    for (int64_t s = s0; s < s1; ++s) {
        double o[VW];
        Vec<OT, VW>::get(O + s * P + p, o);
        const double ws = wt ? wt[s] : 1.0;
#pragma unroll
        for (int q = 0; q < VW; ++q) acc[q] = fma(o[q] - m[q], ws, acc[q]);
    }
#pragma unroll
    for (int q = 0; q < VW; ++q) part[(int64_t)blockIdx.y * P + p + q] = acc[q];
}

// out[p] = scale * sum_c part[c][p] (+ lam * v[p])
__global__ void k_colsum_final(const double *__restrict__ part, int nchunk, int64_t P,
                               double scale, double lam, const double *__restrict__ v,
                               double *__restrict__ out)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    double acc = 0.0;
    for (int c = 0; c < nchunk; ++c) acc += part[(int64_t)c * P + p];
    out[p] = acc * scale + (v ? lam * v[p] : 0.0);
}

// The sum of n <= any block partials, in every thread (the same in every block).
__device__ double sum_parts(const double *part, int n, double *sh)
{
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kThreads) acc += part[i];
    return block_sum(acc, sh);
}

// State of the recursion that the launches of an iteration share.
struct Cg {
    double *x, *r, *p, *ap;
    double *pap_part, *rr_part;   // [nblk] partials of p.Ap and r.r
    int64_t P;
    int nblk, it;
    SrCtl *ctl;

    __host__ __device__ const int *done() const { return &ctl->done[it & 1]; }
};

// For the first launch of iteration g.it > 0: whether an earlier one was the
// last.  `first`: the thread that passes that on to this iteration's launches.
__device__ __forceinline__ bool over(const Cg &g, bool first)
{
    const bool end = g.ctl->done[(g.it - 1) & 1] || g.ctl->stop;
    if (end && first) g.ctl->done[g.it & 1] = 1;
    return end;
}

// beta of iteration g.it > 0 from the previous one's partials of r.r.  r.r of
// the state before iteration i lives in slot i & 1, so a recording block can
// write the new one while the others still read the old one.
__device__ __forceinline__ double beta_of(const Cg &g, double *sh, double &rr)
{
    rr = sum_parts(g.rr_part, g.nblk, sh);
    return rr / g.ctl->rrv[(g.it - 1) & 1];
}

// Records r.r after g.it iterations: ||r|| <= 1e-30 ||F|| is converged far
// beyond FP64 resolution.
__device__ __forceinline__ void record(const Cg &g, double rr, double beta)
{
    g.ctl->rrv[g.it & 1] = rr;
    g.ctl->rr = rr;
    g.ctl->beta = beta;
    g.ctl->it = g.it;
    g.ctl->done[g.it & 1] = !(rr > g.ctl->ff * 1e-60);
}

// First launch of an iteration: u[s] = sum_p (O[s][p] - obar[p]) v[p].  FLY:
// v = r + beta p is formed here element by element (k_ap_small writes it back),
// which saves a launch of 3 to 5 us but reads a third vector per row; else
// v = p.  kRows rows per block, each thread taking VW consecutive elements per
// step (16-byte loads of O); the FP64 vectors are read once per step for all
// the block's rows.  One or two rows are loaded together (a row past the end
// repeats the last); four one after the other, since their loads in one burst
// push the vectors out of the first-level cache (2048 rows of 46,560 floats:
// 75 us against 66, which is 5.8 TB/s).  Each row's sum has the same order
// whatever kRows is.
template <typename OT, int VW, int kRows, bool FLY>
__global__ void __launch_bounds__(kThreads)
k_rowdot(const OT *__restrict__ O, int64_t nrows, const double *__restrict__ obar, Cg g,
         double *__restrict__ u)
{
    __shared__ double sh[kRows][kThreads];
    __shared__ double shb[kThreads];
    if (FLY ? over(g, blockIdx.x == 0 && threadIdx.x == 0) : *g.done() != 0) return;
    const int64_t P = g.P;
    double b = 0.0;
    if (FLY) {
        double rr;
        b = beta_of(g, shb, rr);
        if (blockIdx.x == 0 && threadIdx.x == 0) record(g, rr, b);
        if (!(rr > g.ctl->ff * 1e-60)) return;
    }
    const double *__restrict__ pv = g.p, *__restrict__ rv = g.r;
    const int64_t s0 = (int64_t)blockIdx.x * kRows;
    const OT *row[kRows];
    double acc[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        row[r] = O + min(s0 + r, nrows - 1) * P;
        acc[r] = 0.0;
    }
    for (int64_t p = (int64_t)threadIdx.x * VW; p < P; p += (int64_t)kThreads * VW) {
        double ob[VW], vv[VW], o[kRows][VW];
#pragma unroll
        for (int q = 0; q < VW; ++q) {
            ob[q] = obar[p + q];
            vv[q] = FLY ? fma(b, pv[p + q], rv[p + q]) : pv[p + q];
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            if (kRows > 2 && s0 + r >= nrows) break;
            Vec<OT, VW>::get(row[r] + p, o[r]);
            if (kRows <= 2) continue;
#pragma unroll
            for (int q = 0; q < VW; ++q) acc[r] = fma(o[r][q] - ob[q], vv[q], acc[r]);
        }
        if (kRows > 2) continue;
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int q = 0; q < VW; ++q) acc[r] = fma(o[r][q] - ob[q], vv[q], acc[r]);
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) sh[r][threadIdx.x] = acc[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const double v = tree_sum(sh[r]);
        if (threadIdx.x == 0 && s0 + r < nrows) u[s0 + r] = v;
    }
}

// p = r + beta p as a launch of its own; block 0 records r.r and beta
__global__ void __launch_bounds__(kThreads)
k_update_p(Cg g)
{
    __shared__ double sh[kThreads];
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t k = min(i, g.P - 1);
    const double pi = g.p[k], ri = g.r[k];   // in flight during the sum
    if (over(g, i == 0)) return;
    double rr;
    const double b = beta_of(g, sh, rr);
    if (i < g.P) g.p[i] = fma(b, pi, ri);
    if (blockIdx.x == 0 && threadIdx.x == 0) record(g, rr, b);
}

// launches of the two streaming passes, 16-byte loads when P allows them
template <typename OT>
constexpr int vec_width() { return 16 / (int)sizeof(OT); }

template <typename OT>
void launch_colsum(int64_t nchunk, int64_t P, int n_cu, hipStream_t s, const OT *O, int64_t B,
                   const double *sub, const double *wt, int64_t rpc, double *part,
                   const int *done)
{
    constexpr int VW = vec_width<OT>();
    if (P % VW == 0 && P / (64 * VW) * nchunk >= 2 * n_cu) {
        const dim3 g((unsigned)((P / VW + 63) / 64), (unsigned)nchunk);
        NQS_LAUNCH((k_colsum<OT, VW>), g, dim3(64), 0, s, O, B, P, sub, wt, rpc, part, done);
    } else {
        const dim3 g((unsigned)((P + 63) / 64), (unsigned)nchunk);
        NQS_LAUNCH((k_colsum<OT, 1>), g, dim3(64), 0, s, O, B, P, sub, wt, rpc, part, done);
    }
}

template <typename OT, int ROWS, bool FLY>
void launch_rowdot_r(int64_t nrows, hipStream_t s, const OT *O, const double *obar, const Cg &g,
                     double *u)
{
    constexpr int VW = vec_width<OT>();
    const dim3 grid((unsigned)((nrows + ROWS - 1) / ROWS)), th(kThreads);
    if (g.P % VW == 0)
        NQS_LAUNCH((k_rowdot<OT, VW, ROWS, FLY>), grid, th, 0, s, O, nrows, obar, g, u);
    else
        NQS_LAUNCH((k_rowdot<OT, 1, ROWS, FLY>), grid, th, 0, s, O, nrows, obar, g, u);
}

// Rows a block: four where that leaves two blocks for every CU, else two or one
// (P = 28,064: 1024 rows 32 us with four, 19 with two; 512 rows 20 with two, 14
// with one; 19 us before with four).
template <typename OT>
void launch_rowdot(int64_t nrows, int n_cu, bool fly, hipStream_t s, const OT *O,
                   const double *obar, const Cg &g, double *u)
{
    if (fly && g.it > 0)
        launch_rowdot_r<OT, 1, true>(nrows, s, O, obar, g, u);
    else if (nrows >= (int64_t)8 * n_cu)
        launch_rowdot_r<OT, 4, false>(nrows, s, O, obar, g, u);
    else if (nrows >= (int64_t)4 * n_cu)
        launch_rowdot_r<OT, 2, false>(nrows, s, O, obar, g, u);
    else
        launch_rowdot_r<OT, 1, false>(nrows, s, O, obar, g, u);
}

// partial dot products a.b, one value per block
__global__ void __launch_bounds__(kThreads)
k_dot_part(const double *__restrict__ a, const double *__restrict__ b, int64_t n,
           double *__restrict__ part)
{
    __shared__ double sh[kThreads];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        acc = fma(a[i], b[i], acc);
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// stage 2 of the initial r.r: rr = ff = value; done if ff == 0
__global__ void __launch_bounds__(kThreads)
k_dot_final(const double *__restrict__ part, int nparts, SrCtl *ctl)
{
    __shared__ double sh[kThreads];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += kThreads) acc += part[i];
    acc = block_sum(acc, sh);
    if (threadIdx.x != 0) return;
    ctl->rr = acc;
    ctl->rrv[0] = acc;
    ctl->ff = acc;
    ctl->it = 0;
    ctl->stop = 0;
    ctl->done[0] = !(acc > 0.0);
}

// Ap = scale * sum_c part[c] + lam p, and per block sum p.Ap
__global__ void __launch_bounds__(kThreads)
k_ap_dot(const double *__restrict__ part, int nchunk, double scale, double lam, Cg g)
{
    __shared__ double sh[kThreads];
    if (*g.done()) return;
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double d = 0.0;
    if (i < g.P) {
        double acc = 0.0;
        const double pi = g.p[i];
#pragma unroll 8
        for (int c = 0; c < nchunk; ++c) acc += part[(int64_t)c * g.P + i];
        const double v = fma(acc, scale, lam * pi);
        g.ap[i] = v;
        d = pi * v;
    }
    d = block_sum(d, sh);
    if (threadIdx.x == 0) g.pap_part[blockIdx.x] = d;
}

// k_update_p, k_colsum and k_ap_dot in one (k_rowdot has recorded beta), for P
// up to kSmallP and at most 16 chunks: wave c sums chunk c of 64 columns, the
// first wave adds the chunks in order.  The columns are 16 of each quarter of a
// block of kThreads, so that the first two levels of that block's tree over the
// products p_i (Ap)_i are formed here; the next launch does the rest on the 64
// values a block that go to pap_part (with the products themselves it waited
// 3 us longer for them, every block reading all of them).
constexpr int64_t kSmallP = 16384;
constexpr int kSmallChunks = 16;

template <typename OT>
__global__ void __launch_bounds__(64 * kSmallChunks)
k_ap_small(const OT *__restrict__ O, int64_t B, const double *__restrict__ obar,
           const double *__restrict__ u, int64_t rows_per_chunk, int nchunk, double scale,
           double lam, Cg g)
{
    __shared__ double sh[kSmallChunks][64];
    const int l = threadIdx.x & 63, c = threadIdx.x >> 6;
    const int64_t blk = blockIdx.x >> 2;
    const int m = (blockIdx.x & 3) * 16 + (l & 15);
    const int64_t i = blk * kThreads + (l >> 4) * 64 + m;
    const int64_t k0 = min(i, g.P - 1);
    const double ri = g.r[k0], beta = g.ctl->beta;   // in flight during the sums
    double pi = g.p[k0];
    if (*g.done()) return;
    double acc = 0.0;
    if (i < g.P) {
        const int64_t s0 = (int64_t)c * rows_per_chunk, s1 = min(B, s0 + rows_per_chunk);
        const double m = obar[i];
#pragma unroll 16
        for (int64_t s = s0; s < s1; ++s) acc = fma((double)O[s * g.P + i] - m, u[s], acc);
    }
    sh[c][l] = acc;
    __syncthreads();
    if (c > 0) return;
    double d = 0.0;
    if (i < g.P) {
        double sum = 0.0;
        for (int k = 0; k < nchunk; ++k) sum += sh[k][l];
        if (g.it > 0) {
            pi = fma(beta, pi, ri);
            g.p[i] = pi;
        }
        const double v = fma(sum, scale, lam * pi);
        g.ap[i] = v;
        d = pi * v;
    }
    d += __shfl_down(d, 32, 64);
    d += __shfl_down(d, 16, 64);
    if (l < 16) g.pap_part[blk * 64 + m] = d;
}

// alpha = r.r / p.Ap; x += alpha p, r -= alpha Ap, and per block sum r.r
// (p.Ap <= 0: stop without updating).  SMALL: pap_part holds 64 values a
// block and not the block sums; each wave then forms every fourth block's sum.
template <bool SMALL>
__global__ void __launch_bounds__(kThreads)
k_update_xr(Cg g)
{
    __shared__ double sh[kThreads], sh2[kThreads];
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t k = min(i, g.P - 1);
    const double xi = g.x[k], pi = g.p[k], api = g.ap[k], r0 = g.r[k];   // in flight
    const double rr = g.ctl->rrv[g.it & 1];
    if (*g.done()) return;
    double pap;
    if (SMALL) {
        sh[threadIdx.x] = 0.0;
        __syncthreads();
        const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll 4
        for (int j = w; j < g.nblk; j += 4) {
            double v = g.pap_part[j * 64 + l];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
            if (l == 0) sh[j] = v;
        }
        __syncthreads();
        pap = tree_sum(sh);
    } else {
        pap = sum_parts(g.pap_part, g.nblk, sh);
    }
    if (!(pap > 0.0)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) g.ctl->stop = 1;
        return;
    }
    const double a = rr / pap;
    double acc = 0.0;
    if (i < g.P) {
        g.x[i] = fma(a, pi, xi);
        const double ri = fma(-a, api, r0);
        g.r[i] = ri;
        acc = fma(ri, ri, acc);
    }
    acc = block_sum(acc, sh2);
    if (threadIdx.x == 0) g.rr_part[blockIdx.x] = acc;
    if (blockIdx.x == 0 && threadIdx.x == 0) g.ctl->alpha = a;
}

// x = 0, r = p = F
__global__ void k_init(double *__restrict__ x, double *__restrict__ r, double *__restrict__ p,
                       const double *__restrict__ F, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        x[i] = 0.0;
        r[i] = F[i];
        p[i] = F[i];
    }
}

// mean / variance of e, and d = e - mean
__global__ void __launch_bounds__(1024)
k_center(const double *__restrict__ e, int64_t B, double *__restrict__ d, SrCtl *ctl)
{
    __shared__ double sh[1024];
    double acc = 0.0;
    for (int64_t s = threadIdx.x; s < B; s += 1024) acc += e[s];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 512; off > 0; off >>= 1) {
        if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    const double mean = sh[0] / (double)B;
    __syncthreads();
    acc = 0.0;
    for (int64_t s = threadIdx.x; s < B; s += 1024) {
        const double v = e[s] - mean;
        d[s] = v;
        acc += v * v;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 512; off > 0; off >>= 1) {
        if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        ctl->mean = mean;
        ctl->var = sh[0] / (double)B;
    }
}

// g.it: the iterations asked for; the last one's r.r is not recorded yet
__global__ void __launch_bounds__(kThreads)
k_stats_out(Cg g, double *stats)
{
    __shared__ double sh[kThreads];
    if (g.it > 0 && !over(g, false)) {
        double rr;
        const double b = beta_of(g, sh, rr);
        if (threadIdx.x == 0) record(g, rr, b);
    }
    if (threadIdx.x != 0) return;
    const SrCtl *ctl = g.ctl;
    stats[0] = ctl->mean;
    stats[1] = ctl->var;
    stats[2] = ctl->ff > 0.0 ? sqrt(ctl->rr / ctl->ff) : 0.0;
    stats[3] = (double)ctl->it;
}

struct SrLayout {
    int64_t nchunk, rows_per_chunk, ndot;
    int64_t nblk;   // blocks of kThreads covering P (partials of p.Ap and r.r)
    size_t off_obar, off_F, off_r, off_p, off_ap, off_d, off_u, off_part, off_dot, off_pap,
        off_rrp, off_ctl, total;
};

SrLayout layout(int64_t B, int64_t P)
{
    SrLayout l;
    l.nchunk = std::min<int64_t>(kMaxChunks, std::max<int64_t>(1, (B + 63) / 64));
    l.rows_per_chunk = (B + l.nchunk - 1) / l.nchunk;
    l.ndot = 512;
    l.nblk = std::max<int64_t>(1, (P + kThreads - 1) / kThreads);
    size_t off = 0;
    auto take = [&](size_t n) {
        size_t o = off;
        off += (n * sizeof(double) + 255) & ~(size_t)255;
        return o;
    };
    l.off_obar = take(P);
    l.off_F = take(P);
    l.off_r = take(P);
    l.off_p = take(P);
    l.off_ap = take(P);
    l.off_d = take(B);
    l.off_u = take(B);
    l.off_part = take((size_t)std::max(l.nchunk * P, 64 * l.nblk));   // or k_ap_small's sums
    l.off_dot = take(l.ndot);
    l.off_pap = take(l.nblk);
    l.off_rrp = take(l.nblk);
    l.off_ctl = take(sizeof(SrCtl) / sizeof(double) + 1);
    l.total = off;
    return l;
}

// The rest of an iteration once Ap's partial column sums are in `part`.
void cg_tail(const SrLayout &l, double invB, double lam, const double *part, const Cg &g,
             hipStream_t s)
{
    NQS_LAUNCH(k_ap_dot, dim3(g.nblk), dim3(kThreads), 0, s, part, (int)l.nchunk, invB, lam, g);
    NQS_LAUNCH(k_update_xr<false>, dim3(g.nblk), dim3(kThreads), 0, s, g);
}

Cg state(const SrLayout &l, unsigned char *w, int64_t P, double *x)
{
    Cg g;
    g.x = x;
    g.r = (double *)(w + l.off_r);
    g.p = (double *)(w + l.off_p);
    g.ap = (double *)(w + l.off_ap);
    g.pap_part = (double *)(w + l.off_pap);
    g.rr_part = (double *)(w + l.off_rrp);
    g.P = P;
    g.nblk = (int)l.nblk;
    g.it = 0;
    g.ctl = (SrCtl *)(w + l.off_ctl);
    return g;
}

// x = 0, r = p = F, and r.r
void cg_start(const SrLayout &l, const Cg &g, const double *F, double *dot, hipStream_t s)
{
    const unsigned vgrid = (unsigned)std::min<int64_t>(1024, l.nblk);
    NQS_LAUNCH(k_init, dim3(vgrid), dim3(kThreads), 0, s, g.x, g.r, g.p, F, g.P);
    NQS_LAUNCH(k_dot_part, dim3((unsigned)l.ndot), dim3(kThreads), 0, s, (const double *)g.r,
               (const double *)g.r, g.P, dot);
    NQS_LAUNCH(k_dot_final, dim3(1), dim3(kThreads), 0, s, (const double *)dot, (int)l.ndot,
               g.ctl);
}

template <typename OT>
void sr_solve_t(const OT *O, const double *e, int64_t B, int64_t P, double lam, int n_iter,
                double *x, double *stats, unsigned char *w, int n_cu, hipStream_t s)
{
    const SrLayout l = layout(B, P);
    double *obar = (double *)(w + l.off_obar), *F = (double *)(w + l.off_F);
    double *d = (double *)(w + l.off_d), *u = (double *)(w + l.off_u);
    double *part = (double *)(w + l.off_part), *dot = (double *)(w + l.off_dot);
    Cg g = state(l, w, P, x);
    const unsigned fgrid = (unsigned)l.nblk;
    const double invB = 1.0 / (double)B;

    NQS_LAUNCH(k_center, dim3(1), dim3(1024), 0, s, e, B, d, g.ctl);
    // column means
    launch_colsum<OT>(l.nchunk, P, n_cu, s, O, B, (const double *)nullptr,
                      (const double *)nullptr, l.rows_per_chunk, part, (const int *)nullptr);
    NQS_LAUNCH(k_colsum_final, dim3(fgrid), dim3(kThreads), 0, s, part, (int)l.nchunk, P,
                       invB, 0.0, (const double *)nullptr, obar);
    // F = Obar^T (E - Ebar) / B
    launch_colsum<OT>(l.nchunk, P, n_cu, s, O, B, obar, d, l.rows_per_chunk, part,
                      (const int *)nullptr);
    NQS_LAUNCH(k_colsum_final, dim3(fgrid), dim3(kThreads), 0, s, part, (int)l.nchunk, P,
                       invB, 0.0, (const double *)nullptr, F);
    cg_start(l, g, F, dot, s);
    // (P = 4800, 256 samples: 18.6 us of kernels an iteration against 29; the
    // blocks of the last launch read P / 4 values each, hence the line at 16 K)
    const bool small = P <= kSmallP && l.nchunk <= kSmallChunks;
    if (small) g.pap_part = part;
    for (; g.it < n_iter; ++g.it) {
        // Ap = Obar^T (Obar p) / B + lambda p
        if (!small && g.it > 0) NQS_LAUNCH(k_update_p, dim3(fgrid), dim3(kThreads), 0, s, g);
        launch_rowdot<OT>(B, n_cu, small, s, O, obar, g, u);
        if (small) {
            NQS_LAUNCH(k_ap_small<OT>, dim3(4 * fgrid),
                       dim3(64 * (unsigned)l.nchunk), 0, s, O, B, (const double *)obar,
                       (const double *)u, l.rows_per_chunk, (int)l.nchunk, invB, lam, g);
            NQS_LAUNCH(k_update_xr<true>, dim3(fgrid), dim3(kThreads), 0, s, g);
        } else {
            launch_colsum<OT>(l.nchunk, P, n_cu, s, O, B, obar, u, l.rows_per_chunk, part,
                              g.done());
            cg_tail(l, invB, lam, part, g, s);
        }
    }
    if (stats) NQS_LAUNCH(k_stats_out, dim3(1), dim3(kThreads), 0, s, g, stats);
}

// The same solve with O never held whole: rows [r0, r0 + nb) of O are
// produced on demand into a buffer of `chunk` rows by `rows` (which recomputes
// them from the samples).  chunk is a multiple of the reduction row block, so
// each block's partial column sums see exactly the rows, in exactly the order,
// of the stored-O solve, and the results are the same bit for bit.  One pass
// over O needs nc = ceil(B / chunk) chunks; a pass starts with the chunk left
// in the buffer by the previous one, so an iteration recomputes 2 (nc - 1)
// chunks.
template <typename OT>
void sr_solve_rows_t(const SrRows &rows, OT *obuf, int64_t chunk, const double *e, int64_t B,
                     int64_t P, double lam, int n_iter, double *x, double *stats,
                     unsigned char *w, int n_cu, hipStream_t s)
{
    const SrLayout l = layout(B, P);
    double *obar = (double *)(w + l.off_obar), *F = (double *)(w + l.off_F);
    double *d = (double *)(w + l.off_d), *u = (double *)(w + l.off_u);
    double *part = (double *)(w + l.off_part), *dot = (double *)(w + l.off_dot);
    Cg g = state(l, w, P, x);
    const int64_t rpc = l.rows_per_chunk;
    const int64_t nc = (B + chunk - 1) / chunk;
    const unsigned fgrid = (unsigned)l.nblk;
    const double invB = 1.0 / (double)B;
    int64_t resident = -1;   // chunk whose rows are in obuf

    // one pass over all chunks: fn(r0, nb) sees rows [r0, r0 + nb) in obuf
    auto pass = [&](auto &&fn) {
        int64_t order0 = resident >= 0 ? resident : 0;
        for (int64_t i = 0; i < nc; ++i) {
            const int64_t ci = (order0 + i) % nc;
            const int64_t r0 = ci * chunk;
            const int nb = (int)std::min<int64_t>(chunk, B - r0);
            if (ci != resident) {
                rows(r0, nb, obuf, s);
                resident = ci;
            }
            fn(r0, nb);
        }
    };
    // partial column sums of rows [r0, r0 + nb) into their reduction blocks
    auto colsum = [&](int64_t r0, int nb, const double *sub, const double *wt, const int *done) {
        launch_colsum<OT>((nb + rpc - 1) / rpc, P, n_cu, s, (const OT *)obuf, (int64_t)nb, sub,
                          wt ? wt + r0 : wt, rpc, part + (r0 / rpc) * P, done);
    };

    NQS_LAUNCH(k_center, dim3(1), dim3(1024), 0, s, e, B, d, g.ctl);
    pass([&](int64_t r0, int nb) {
        colsum(r0, nb, (const double *)nullptr, (const double *)nullptr, (const int *)nullptr);
    });
    NQS_LAUNCH(k_colsum_final, dim3(fgrid), dim3(kThreads), 0, s, part, (int)l.nchunk, P, invB,
               0.0, (const double *)nullptr, obar);
    pass([&](int64_t r0, int nb) { colsum(r0, nb, obar, d, (const int *)nullptr); });
    NQS_LAUNCH(k_colsum_final, dim3(fgrid), dim3(kThreads), 0, s, part, (int)l.nchunk, P, invB,
               0.0, (const double *)nullptr, F);
    cg_start(l, g, F, dot, s);
    for (; g.it < n_iter; ++g.it) {
        if (g.it > 0) NQS_LAUNCH(k_update_p, dim3(fgrid), dim3(kThreads), 0, s, g);
        pass([&](int64_t r0, int nb) {
            launch_rowdot<OT>(nb, n_cu, false, s, (const OT *)obuf, obar, g, u + r0);
        });
        pass([&](int64_t r0, int nb) { colsum(r0, nb, obar, u, g.done()); });
        cg_tail(l, invB, lam, part, g, s);
    }
    if (stats) NQS_LAUNCH(k_stats_out, dim3(1), dim3(kThreads), 0, s, g, stats);
}

}  // namespace

size_t sr_workspace_bytes(int64_t B, int64_t P) { return layout(B, P).total; }

void launch_sr_solve(const void *O, nqs_dtype odt, const double *e_loc, int64_t B, int64_t P,
                     double lambda, int n_iter, double *x, double *stats, void *work,
                     int n_cu, hipStream_t s)
{
    if (odt == NQS_FP32)
        sr_solve_t<float>((const float *)O, e_loc, B, P, lambda, n_iter, x, stats,
                          (unsigned char *)work, n_cu, s);
    else
        sr_solve_t<double>((const double *)O, e_loc, B, P, lambda, n_iter, x, stats,
                           (unsigned char *)work, n_cu, s);
}

int64_t sr_row_block(int64_t B) { return layout(B, 1).rows_per_chunk; }

void launch_sr_solve_rows(const SrRows &rows, void *obuf, int64_t chunk, nqs_dtype odt,
                          const double *e_loc, int64_t B, int64_t P, double lambda, int n_iter,
                          double *x, double *stats, void *work, int n_cu, hipStream_t s)
{
    if (odt == NQS_FP32)
        sr_solve_rows_t<float>(rows, (float *)obuf, chunk, e_loc, B, P, lambda, n_iter, x, stats,
                               (unsigned char *)work, n_cu, s);
    else
        sr_solve_rows_t<double>(rows, (double *)obuf, chunk, e_loc, B, P, lambda, n_iter, x,
                                stats, (unsigned char *)work, n_cu, s);
}

}  // namespace nqs

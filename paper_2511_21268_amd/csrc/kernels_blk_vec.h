// Element-wise, transfer, coarsest-level and reduction kernels of the 16-column
// block solve (row-major N x 16 vectors; the matrix passes are in kernels_blk.h).
#pragma once
#include "kernels.h"

namespace amgk {

constexpr int NB = 16;

// per-column scalar slots: sc[slot * NB + j]
enum BSlot { B_RZ = 0, B_PQ, B_RR, B_ALPHA, B_BETA, B_PR, B_ZQ, B_FF, B_FLAG, B_DONE, B_ITERS, B_THR, B_NSLOTS };
enum BFin { BF_FF = 0, BF_RR0, BF_RZ0, BF_PQ_CG, BF_PQ_FCG, BF_RR, BF_RZ_CG, BF_ZQ_FCG };

__device__ inline bool bactive(const double *sc, int j) { return sc[B_DONE * NB + j] == 0.0 && sc[B_FLAG * NB + j] == 0.0; }

// ---- elementwise block kernels (one thread per row, 16 columns) ---------------

template <typename VT, typename FT>
__global__ void k_scale_blk(int64_t n, const VT *__restrict__ invd, const FT *__restrict__ f, VT *__restrict__ u,
                            VT coef)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const VT di = invd[i];
#pragma unroll
    for (int j = 0; j < NB; j++) u[i * NB + j] = coef * (di * (VT)f[i * NB + j]);
}

// Restriction of 16 columns, one element (coarse row I, column j) per thread:
// consecutive threads on consecutive addresses, the members read together.
// coef == 1 keeps the l1 sweep's bits: 1 * (d * f) == d * f exactly.
template <typename VT>
__global__ __launch_bounds__(256) void k_restrict_blk(int64_t nc, int mw, const int32_t *__restrict__ members,
                                                      const VT *__restrict__ pc, const VT *__restrict__ r,
                                                      VT *__restrict__ fc, const VT *__restrict__ invdc,
                                                      VT *__restrict__ uc, VT coef)
{
#pragma clang fp contract(off)
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, I = e / NB;
    const int j = (int)(e % NB);
    if (I >= nc) return;
    constexpr int MW = 8;
    int m[MW];
    VT p[MW], v[MW];
#pragma unroll
    for (int t = 0; t < MW; t++) m[t] = t < mw ? members[I * mw + t] : -1;
#pragma unroll
    for (int t = 0; t < MW; t++) {
        const int64_t i = m[t] < 0 ? 0 : m[t];
        if (t < mw) { p[t] = pc[i]; v[t] = r[i * NB + j]; }
    }
    VT s = 0;
#pragma unroll
    for (int t = 0; t < MW; t++)
        if (m[t] >= 0) {
            VT prod = p[t] * v[t];
            s = s + prod;
        }
    fc[e] = s;
    if (uc) uc[e] = coef * (invdc[I] * s);
}

template <typename VT>
__global__ void k_prolong_blk(int64_t n, const int32_t *__restrict__ agg, const VT *__restrict__ pc,
                              const VT *__restrict__ e, VT *__restrict__ u)
{
#pragma clang fp contract(off)
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const VT pi = pc[i];
    const int64_t a = (int64_t)agg[i] * NB;
#pragma unroll
    for (int j = 0; j < NB; j++) {
        VT prod = pi * e[a + j];
        u[i * NB + j] = u[i * NB + j] + prod;
    }
}

template <typename VT, typename OT>
__global__ void k_add_blk(int64_t n, const VT *__restrict__ x, const VT *__restrict__ c, OT *__restrict__ y)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * NB) return;
    y[i] = (OT)(x[i] + c[i]);
}

// Coarsest level for 16 columns, one of the two products of k_coarse_solve per
// launch: LOWER Y = L^{-1} F (M: the transposed inverse factor), else E = L^{-T} Y
// (M: the inverse factor; Y: global scratch, n x 16).  One element (row i, column
// j) per thread in k_coarse_solve's segments and order, so each column equals its
// result.  The rows of F and the block's columns of M come through LDS, 64 of
// each segment at a time: one thread per element reading them from memory
// waited a latency every few terms.
constexpr int CBLK_ROWS = 256 / NB, CBLK_K = 64;
template <bool LOWER, typename FT, typename ET>
__global__ __launch_bounds__(256) void k_coarse_product_blk(int n, int ld, const double *__restrict__ M,
                                                            const FT *__restrict__ f, ET *__restrict__ e)
{
    __shared__ double fs[COARSE_SEGS * CBLK_K][NB], ms[COARSE_SEGS * CBLK_K][CBLK_ROWS + 1];
    const int j = threadIdx.x & (NB - 1), r = threadIdx.x / NB, i0 = blockIdx.x * CBLK_ROWS;
    const int len = coarse_len(n);
    // the terms of the block's rows; M is zero in the rest of its square
    const int ka = LOWER ? 0 : i0, kb = LOWER ? min(i0 + CBLK_ROWS, n) : n;
    double s[COARSE_SEGS];
#pragma unroll
    for (int q = 0; q < COARSE_SEGS; q++) s[q] = 0.0;
    for (int c = 0; c < len; c += CBLK_K) {
        __syncthreads();
        // row h of the tiles: k = q len + c + t (zeros past the segment)
#pragma unroll
        for (int g = 0; g < COARSE_SEGS * CBLK_K / CBLK_ROWS; g++) {
            const int h = g * CBLK_ROWS + r, q = h / CBLK_K, t = c + h % CBLK_K, k = q * len + t;
            const bool live = t < len && k >= ka && k < kb;
            fs[h][j] = live ? (double)f[(int64_t)k * NB + j] : 0.0;
            ms[h][j] = live && i0 + j < n ? M[(int64_t)k * ld + i0 + j] : 0.0;
        }
        __syncthreads();
        const int steps = min(CBLK_K, len - c);
        for (int t = 0; t < steps; t++)
#pragma unroll
            for (int q = 0; q < COARSE_SEGS; q++) {
                const int k = q * len + c + t;
                if (k >= ka && k < kb) s[q] = fma(ms[q * CBLK_K + t][r], fs[q * CBLK_K + t][j], s[q]);
            }
    }
    if (i0 + r < n) e[(int64_t)(i0 + r) * NB + j] = (ET)((s[0] + s[1]) + (s[2] + s[3]));
}

// the same sum for one element in one thread (V-cycle tail of 16 columns)
template <bool LOWER, typename FT>
__device__ __forceinline__ double coarse_row_blk(int n, int ld, const double *__restrict__ M, const FT *__restrict__ f,
                                                 int i, int j)
{
    const int len = coarse_len(n);
    double s[COARSE_SEGS];
#pragma unroll
    for (int q = 0; q < COARSE_SEGS; q++) {
        s[q] = 0.0;
        const int k0 = LOWER ? q * len : max(q * len, i), k1 = min((q + 1) * len, LOWER ? i + 1 : n);
#pragma unroll 8
        for (int k = k0; k < k1; k++) s[q] = fma(M[(int64_t)k * ld + i], (double)f[(int64_t)k * NB + j], s[q]);
    }
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// Column-major (n x k, leading dimension n) <-> row-major block (n x NB).
static __global__ void k_pack_blk(int64_t n, int k, const double *__restrict__ cm, double *__restrict__ rm)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
#pragma unroll
    for (int j = 0; j < NB; j++) rm[i * NB + j] = j < k ? cm[(int64_t)j * n + i] : 0.0;
}

static __global__ void k_unpack_blk(int64_t n, int k, const double *__restrict__ rm, double *__restrict__ cm)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    for (int j = 0; j < k; j++) cm[(int64_t)j * n + i] = rm[i * NB + j];
}

// ---- element-parallel block vector kernels ----------------------------------
//
// Thread t of the grid handles the elements e = t, t + T, ... (T = threads in
// the grid, a multiple of 16) of the row-major N x 16 arrays, so a wave's load
// is 64 consecutive values and every thread keeps one column j = e % 16.  Dot
// partials per column: the thread's running sum, the 4 lanes of each column in
// a wave (butterfly over lane bits 4 and 5), then the block's waves in order:
// partial[(2 * blockIdx.x + d) * NB + j].

__device__ inline void blk_col_partials(double s0, double s1, double *lds /* 2 * 4 * NB */, double *partial)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    s0 += __shfl_xor(s0, 16, 64);
    s0 += __shfl_xor(s0, 32, 64);
    s1 += __shfl_xor(s1, 16, 64);
    s1 += __shfl_xor(s1, 32, 64);
    if (lane < NB) {
        lds[wid * NB + lane] = s0;
        lds[(4 + wid) * NB + lane] = s1;
    }
    __syncthreads();
    if (threadIdx.x < NB) {
        const int j = threadIdx.x;
        partial[(2 * blockIdx.x) * NB + j] = ((lds[j] + lds[NB + j]) + lds[2 * NB + j]) + lds[3 * NB + j];
        partial[(2 * blockIdx.x + 1) * NB + j] =
            ((lds[4 * NB + j] + lds[5 * NB + j]) + lds[6 * NB + j]) + lds[7 * NB + j];
    }
}

// per-column partials of (a, b) and (a, c) (c may be NULL)
static __global__ __launch_bounds__(256) void k_dot2_blk(int64_t n, const double *__restrict__ a, const double *__restrict__ b,
                                                  const double *__restrict__ c, double *__restrict__ partial)
{
    __shared__ double lds[8 * NB];
    double s0 = 0.0, s1 = 0.0;
    const int64_t m = n * NB;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < m; e += (int64_t)gridDim.x * 256) {
        s0 = fma(a[e], b[e], s0);
        if (c) s1 = fma(a[e], c[e], s1);
    }
    blk_col_partials(s0, s1, lds, partial);
}

// u += alpha p ; r -= alpha q for the active columns; partials of (r, r); with
// u0 the first smoothing step of the next V-cycle from zero, coef D^{-1} r (every
// column), whose kernel it saves.
template <typename VT>
__global__ __launch_bounds__(256) void k_bcg_update(int64_t n, const double *__restrict__ sc, double *__restrict__ u,
                                                    double *__restrict__ r, const double *__restrict__ p,
                                                    const double *__restrict__ q, double *__restrict__ partial,
                                                    const VT *__restrict__ invd, VT *__restrict__ u0, VT coef)
{
    __shared__ double lds[8 * NB];
    const int j = threadIdx.x & (NB - 1);
    const bool act = bactive(sc, j);
    const double al = sc[B_ALPHA * NB + j];
    double s = 0.0;
    const int64_t m = n * NB;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < m; e += (int64_t)gridDim.x * 256) {
        double ri = r[e];
        if (act) {
            u[e] = fma(al, p[e], u[e]);
            ri = fma(-al, q[e], ri);
            r[e] = ri;
        }
        if (u0) u0[e] = coef * (invd[e / NB] * (VT)ri);
        s = fma(ri, ri, s);
    }
    blk_col_partials(s, 0.0, lds, partial);
}

// p = z + beta p for the active columns
static __global__ __launch_bounds__(256) void k_bcg_pupdate(int64_t n, const double *__restrict__ sc,
                                                     const double *__restrict__ z, double *__restrict__ p)
{
    const int j = threadIdx.x & (NB - 1);
    if (!bactive(sc, j)) return;
    const double be = sc[B_BETA * NB + j];
    const int64_t m = n * NB;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < m; e += (int64_t)gridDim.x * 256)
        p[e] = fma(be, p[e], z[e]);
}

// First stage of k_bfinalize for many partials: the strided sums that its
// thread t would form (partials t, t + FIN_THREADS, ... in ascending order),
// one grid thread per (t, dot, column): strided[(d * NB + j) * FIN_THREADS + t].
static __global__ __launch_bounds__(256) void k_bfin_strided(const double *__restrict__ partial, int nblk,
                                                      double *__restrict__ strided)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;   // < 2 * NB * FIN_THREADS
    const int j = idx % NB, d = (idx / NB) % 2, t = idx / (2 * NB);
    double s = 0.0;
    for (int b = t; b < nblk; b += FIN_THREADS) s += partial[(2 * b + d) * NB + j];
    strided[(d * NB + j) * FIN_THREADS + t] = s;
}

// Final per-column sums of the partials (index order) and the scalar
// recurrences, masks and iteration counters of the 16 independent solves: block
// j takes column j (one block for all columns spent 28 us in 32 butterflies
// per wave).  A partial's 16 columns share a cache line, so a block reads every
// line of the dots it takes: 4,096 partials 6 us with the first dot's lines
// alone, the loads before the sums; 9 us with both dots' always read.  With strided != nullptr the
// per-thread strided sums come from k_bfin_strided (the same values).  host
// (mapped, may be NULL): the column's flags, which the host's stopping test
// reads, written there directly.
static __global__ __launch_bounds__(FIN_THREADS) void k_bfinalize(const double *__restrict__ partial, int nblk,
                                                                  double *sc, int op, double tol,
                                                                  const double *__restrict__ strided, double *host)
{
    // the order of k_finalize: thread strides, butterfly, waves in order
    constexpr int NW = FIN_THREADS / 64;
    __shared__ double lds[2 * NW];
    const int j = blockIdx.x, t = threadIdx.x;
    const bool two = op == BF_PQ_FCG;   // the only one that takes both dots
    double s0 = 0.0, s1 = 0.0;
    if (strided) {
        s0 = strided[j * FIN_THREADS + t];
        if (two) s1 = strided[(NB + j) * FIN_THREADS + t];
    } else {
        // at most four partials a thread (bfinalize), all loaded before the sums
        double v0[4], v1[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int b = t + u * FIN_THREADS;
            v0[u] = b < nblk ? partial[(2 * b) * NB + j] : 0.0;
            v1[u] = two && b < nblk ? partial[(2 * b + 1) * NB + j] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (t + u * FIN_THREADS < nblk) { s0 += v0[u]; s1 += v1[u]; }
    }
    const double a = block_sum_n<NW>(s0, lds), b = two ? block_sum_n<NW>(s1, lds + NW) : 0.0;
    if (t != 0) return;
    {
        double *F = sc + B_FLAG * NB + j, *D = sc + B_DONE * NB + j;
        switch (op) {
        case BF_FF:
            sc[B_FF * NB + j] = a;
            sc[B_THR * NB + j] = tol * sqrt(a);
            break;
        case BF_RR0:   // initial residual: converged columns are done before any update
            sc[B_RR * NB + j] = a;
            if (sc[B_FF * NB + j] == 0.0 || sqrt(a) <= sc[B_THR * NB + j]) *D = 1.0;
            break;
        case BF_RZ0:
            if (*D != 0.0) break;
            sc[B_RZ * NB + j] = a;
            if (!(a > 0.0) || !isfinite(a)) *F = 2.0;
            break;
        case BF_PQ_CG:
        case BF_PQ_FCG:
            if (*D != 0.0 || *F != 0.0) break;
            sc[B_PQ * NB + j] = a;
            if (op == BF_PQ_FCG) sc[B_PR * NB + j] = b;
            if (!(a > 0.0) || !isfinite(a)) *F = 1.0;
            else sc[B_ALPHA * NB + j] = (op == BF_PQ_FCG ? b : sc[B_RZ * NB + j]) / a;
            break;
        case BF_RR:   // one more completed update of this column
            if (*D != 0.0 || *F != 0.0) break;
            sc[B_RR * NB + j] = a;
            sc[B_ITERS * NB + j] += 1.0;
            if (sqrt(a) <= sc[B_THR * NB + j]) *D = 1.0;
            break;
        case BF_RZ_CG:
            if (*D != 0.0 || *F != 0.0) break;
            if (!(a > 0.0) || !isfinite(a)) *F = 2.0;
            else { sc[B_BETA * NB + j] = a / sc[B_RZ * NB + j]; sc[B_RZ * NB + j] = a; }
            break;
        case BF_ZQ_FCG:
            if (*D != 0.0 || *F != 0.0) break;
            sc[B_ZQ * NB + j] = a;
            if (!isfinite(a)) *F = 2.0;
            else sc[B_BETA * NB + j] = -a / sc[B_PQ * NB + j];
            break;
        }
        if (host) {
            host[B_DONE * NB + j] = *D;
            host[B_FLAG * NB + j] = *F;
        }
    }
}

}  // namespace amgk

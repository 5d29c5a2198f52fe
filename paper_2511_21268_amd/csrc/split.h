// Matrix passes with W wavefronts per slice (W = 4 or 8), for images of too few
// slices to fill the GPU with one wavefront each.
//
// What bounds k_sell there is a serial chain of memory latencies, not
// bandwidth: one wave walks a slice in steps of 8 or 16 entries per row and
// waits for each (36k rows of 729 entries, 210 MB: 92 us, 2.3 TB/s; a 4,300-row
// coarse level: 15 us for 4 MB).  Here a block of W waves takes the slice in turns
// of T entries per row: every wave has the values, columns and x of its next
// turn in flight (64 rows wide, the loads of the one-wave walk) while the
// others take theirs.
//
// The sum itself stays the sequential chain of the one-wave walk, so that
// every result keeps its bits (the block, tail and window kernels and the FP32
// V-cycle are compared with it bit for bit): the rows' partial sums go from
// wave to wave through LDS, one block barrier per turn.  A turn is about 500
// cycles (T = 32: 32 dependent FMAs, an LDS write and read, the barrier),
// 2 us for 330 entries, below what the loads took.
//
// Measured, kernel times, one wave per slice against this: SpMV of 36k rows of
// 729 entries 92 -> 44 us (2.3 -> 4.7 TB/s); FP32 residual of 33k rows of 1,331 entries
// 98 -> 52 us, of its coarse levels (129, 33, 9 slices) 67, 39, 22 -> 29, 16, 9
// us; the V-cycle of that system 365 -> 180 us.  Now a pass is bound by the
// loads in flight: in FP64 near HBM's rate from about 500 slices on, in FP32 half
// as many bytes a wave (2.6 TB/s at 512 slices, of whose 52 us the turns are 9),
// with fewer slices by their latency.
//
// After the last turn wave 0 runs the epilogue of k_sell on the sums, one lane
// per row, dot partials included; it asked for the epilogue's operands first.
#pragma once
#include "cheb.h"

namespace amgk {

constexpr int TURN = 32;   // entries per row and turn (values and x in registers: 128 VGPRs in FP64)

// sums[r] = (K x)_{row r of slice s}; all W waves of the block call it.
template <int W, typename VT, typename IT>
__device__ __forceinline__ void split_rows(const Sell<VT, IT> &A, int64_t s, int lane, int wid,
                                           const VT *__restrict__ x, VT *sums)
{
    constexpr int T = TURN, TG = T / 8;   // groups of 8 entries per turn
    const int64_t base = A.soff[s];
    const int ng = (int)((A.soff[s + 1] - base) / (8 * SLICE)), nt = (ng + TG - 1) / TG;
    const int64_t ib = A.ibase[s];
    if (nt == 0) {
        if (wid == 0) sums[lane] = 0;
        lds_barrier();
        return;
    }
    VT v[T], xv[T];
    // fetch(t): the index data of turn t, asked for a whole round of turns
    // before columns(t, c) makes columns of it, so that no wave waits for it
    // between two barriers.  Groups past the last one are loaded from it and
    // take no part in the sums.
    auto walk = [&](auto fetch, auto columns) {
        auto load = [&](int t) {
            int c[T];
            columns(t, c);
#pragma unroll
            for (int g = 0; g < TG; g++) {
                VT o[8];
                load8c<SLICE>(A.val, base, 8 * min(t * TG + g, ng - 1), lane, o);
#pragma unroll
                for (int k = 0; k < 8; k++) v[8 * g + k] = o[k];
            }
#pragma unroll
            for (int k = 0; k < T; k++) xv[k] = ld32(x, c[k]);
            fetch(min(t + W, nt - 1));
        };
        fetch(min(wid, nt - 1));
        if (wid < nt) load(wid);
        for (int t = 0; t < nt; t++) {
            const bool mine = t % W == wid;
            if (mine) {
                VT acc = t == 0 ? (VT)0 : sums[lane];
#pragma unroll
                for (int g = 0; g < TG; g++)
                    if (t * TG + g < ng)
#pragma unroll
                        for (int k = 0; k < 8; k++) acc = fma(v[8 * g + k], xv[8 * g + k], acc);
                sums[lane] = acc;
            }
            lds_barrier();
            if (mine && t + W < nt) load(t + W);
        }
    };
    if (ib < 0) {
        // shared offsets: read through the scalar cache
        const int64_t e = -1 - ib;
        const int32_t *so = A.shoff + (e >> 1);
        const int row = (int)(s * SLICE) + lane, hi = (int)A.ncols - 1;
        const bool clamp = !(e & 1);
        walk([](int) {},
             [&](int t, int (&c)[T]) {
#pragma unroll
                 for (int k = 0; k < T; k++) {
                     c[k] = row + so[8 * min(t * TG + k / 8, ng - 1) + k % 8];
                     if (clamp) c[k] = min(max(c[k], 0), hi);
                 }
             });
    } else if constexpr (sizeof(IT) == 2) {
        // 16-bit deltas: a turn starts from the column before its first group
        vu4 raw[TG];
        int first = 0;
        walk(
            [&](int t) {
                first = A.gcol[ib / 8 + (int64_t)(t * TG) * SLICE + lane];
#pragma unroll
                for (int g = 0; g < TG; g++)
                    raw[g] = __builtin_nontemporal_load(reinterpret_cast<const vu4 *>(A.idx + ib) +
                                                        (int64_t)min(t * TG + g, ng - 1) * SLICE + lane);
            },
            [&](int t, int (&c)[T]) {
                int col = first;
#pragma unroll
                for (int g = 0; g < TG; g++) {
                    const bool live = t * TG + g < ng;
#pragma unroll
                    for (int k = 0; k < 8; k++) {
                        const unsigned w = raw[g][k / 2];
                        if (live) col += (int)(k % 2 ? w >> 16 : w & 0xffffu);
                        c[8 * g + k] = col;
                    }
                }
            });
    } else {
        vi4 raw[2 * TG];
        walk(
            [&](int t) {
#pragma unroll
                for (int g = 0; g < 2 * TG; g++)
                    raw[g] = __builtin_nontemporal_load(reinterpret_cast<const vi4 *>(A.idx + ib) +
                                                        (int64_t)min(t * 2 * TG + g, 2 * ng - 1) * SLICE + lane);
            },
            [&](int, int (&c)[T]) {
#pragma unroll
                for (int k = 0; k < T; k++) c[k] = raw[k / 4][k % 4];
            });
    }
}

// k_sell with W waves per slice: block s takes slice s.
template <typename VT, typename FT, typename OT, typename IT, int EPI, int NDOT, int W>
__global__ __launch_bounds__(SLICE *W) void k_split(const Sell<VT, IT> A, const VT *__restrict__ x,
                                                    const FT *__restrict__ f, const VT *__restrict__ invd,
                                                    OT *__restrict__ y, const double *__restrict__ g0,
                                                    const double *__restrict__ g1, double *__restrict__ partial,
                                                    VT coef)
{
    __shared__ VT sums[SLICE];
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int64_t s = blockIdx.x;
    // wave 0 asks for the epilogue's operands first
    int64_t row = -1;
    RowOps<VT, FT, EPI, NDOT> ops;
    if (wid == 0) {
        row = A.row_of(s * SLICE + lane);
        if (row >= 0) ops.load(row, x, f, invd, g0, g1);
    }
    split_rows<W>(A, s, lane, wid, x, sums);
    if (wid != 0) return;
    double d0 = 0.0, d1 = 0.0;
    if (row >= 0) y[row] = ops.template finish<OT>(sums[lane], coef, d0, d1);
    if (NDOT >= 1) {
        const double t0 = wave_sum(d0), t1 = NDOT >= 2 ? wave_sum(d1) : 0.0;
        if (lane == 0) {
            partial[2 * s] = t0;
            partial[2 * s + 1] = t1;
        }
    }
}

// k_sell_post with W waves per slice.
template <typename VT, typename OT, typename IT, int NDOT, int W>
__global__ __launch_bounds__(SLICE *W) void k_split_post(const Sell<VT, IT> A, const VT *__restrict__ e,
                                                         const VT *__restrict__ u, const VT *__restrict__ r,
                                                         const VT *__restrict__ invd, const int32_t *__restrict__ agg,
                                                         const VT *__restrict__ pc, OT *__restrict__ y,
                                                         const double *__restrict__ g0, double *__restrict__ partial)
{
    __shared__ VT sums[SLICE];
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int64_t s = blockIdx.x;
    int64_t row = -1;
    VT ur = 0, pr = 0, er = 0, dr = 0, rr = 0;
    double g = 0.0;
    if (wid == 0) {
        row = A.row_of(s * SLICE + lane);
        if (row >= 0) {
            er = e[agg[row]];
            ur = u[row]; pr = pc[row]; dr = invd[row]; rr = r[row];
            if (NDOT >= 1) g = g0[row];
        }
    }
    split_rows<W>(A, s, lane, wid, e, sums);
    if (wid != 0) return;
    double d0 = 0.0;
    if (row >= 0) {
        const VT out = post_update(ur, pr, er, dr, rr, sums[lane]);
        y[row] = (OT)out;
        if (NDOT >= 1) d0 = (double)out * g;
    }
    if (NDOT >= 1) {
        const double t0 = wave_sum(d0);
        if (lane == 0) {
            partial[2 * s] = t0;
            partial[2 * s + 1] = 0.0;
        }
    }
}

// k_sell_post_res with W waves per slice.
template <typename VT, typename IT, int W>
__global__ __launch_bounds__(SLICE *W) void k_split_post_res(const Sell<VT, IT> A, const VT *__restrict__ e,
                                                             const VT *__restrict__ u, VT *__restrict__ r,
                                                             const int32_t *__restrict__ agg,
                                                             const VT *__restrict__ pc, VT *__restrict__ y)
{
    __shared__ VT sums[SLICE];
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int64_t s = blockIdx.x;
    int64_t row = -1;
    VT ur = 0, pr = 0, er = 0, rr = 0;
    if (wid == 0) {
        row = A.row_of(s * SLICE + lane);
        if (row >= 0) {
            er = e[agg[row]];
            ur = u[row]; pr = pc[row]; rr = r[row];
        }
    }
    split_rows<W>(A, s, lane, wid, e, sums);
    if (wid != 0 || row < 0) return;
    y[row] = ur + pr * er;
    r[row] = rr - sums[lane];
}

// k_sell_cheb with W waves per slice.
template <typename IT, int MODE, int W>
__global__ __launch_bounds__(SLICE *W) void k_split_cheb(const Sell<double, IT> A, const double *__restrict__ x,
                                                         const double *__restrict__ f, double *__restrict__ r,
                                                         const double *__restrict__ invd, double *__restrict__ u,
                                                         double *__restrict__ dn, double a, double b, int first)
{
    __shared__ double sums[SLICE];
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int64_t s = blockIdx.x;
    int64_t row = -1;
    ChebRow<MODE> ops;
    if (wid == 0) {
        row = A.row_of(s * SLICE + lane);
        if (row >= 0) ops.load(row, x, f, r, invd, u, first);
    }
    split_rows<W>(A, s, lane, wid, x, sums);
    if (wid != 0 || row < 0) return;
    ops.finish(row, sums[lane], r, u, dn, a, b, first);
}

}  // namespace amgk

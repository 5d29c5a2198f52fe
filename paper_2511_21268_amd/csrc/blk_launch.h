// Launchers of the 16-column matrix passes (kernels_blk.h).  Each kernel
// family is compiled in a translation unit of its own (blk_*.hip), for the
// combinations of types, epilogue and dots that the block V-cycle and the
// Krylov loops use (BLK_PASSES).
#pragma once
#include <algorithm>

#include "devmat.h"

namespace amgk {

// What a block pass is launched with: the context's stream, variant and partials.
struct BlkCfg {
    hipStream_t stream;
    int win, share;      // staged windows: rows per lane (0: off), shared-window mask
    int lpr, threads;    // lanes per row and threads per block of the other images
    double *partial;
};

template <typename VT, typename FT, typename OT> struct BlkVecs {
    const VT *x;
    const FT *f;
    const VT *invd;
    OT *y;
    const double *g0, *g1;
    VT coef;
};

// Operands of the fused prolongation + post-smoothing.
template <typename VT, typename OT> struct PostVecs {
    const VT *e, *u, *r, *invd;
    const int32_t *agg;
    const VT *pc;
    OT *y;
    const double *g0;
};

// (VT, FT, OT, EPI, NDOT) of the block passes
#define BLK_PASSES(X)                          \
    X(double, double, double, EPI_SPMV, 0)     \
    X(double, double, double, EPI_SPMV, 1)     \
    X(double, double, double, EPI_SPMV, 2)     \
    X(double, double, double, EPI_RESID, 0)    \
    X(float, double, float, EPI_RESID, 0)      \
    X(float, float, float, EPI_RESID, 0)       \
    X(double, double, double, EPI_SMOOTH, 0)   \
    X(double, double, double, EPI_SMOOTH, 1)   \
    X(float, double, float, EPI_SMOOTH, 0)     \
    X(float, double, double, EPI_SMOOTH, 0)    \
    X(float, double, double, EPI_SMOOTH, 1)    \
    X(float, float, float, EPI_SMOOTH, 0)      \
    X(double, double, double, EPI_POLY, 0)     \
    X(float, double, float, EPI_POLY, 0)       \
    X(float, float, float, EPI_POLY, 0)

#define BLK_DECL(FN)                                            \
    template <typename VT, typename FT, typename OT, int EPI, int NDOT> \
    unsigned FN(const BlkCfg &c, const DevMat &A, const BlkVecs<VT, FT, OT> &v)
// each returns the number of dot-partial blocks
BLK_DECL(blk_win);    // windows per wave
BLK_DECL(blk_wins);   // windows shared by the waves of a block
BLK_DECL(blk_rows);   // c.lpr lanes per row on a SELL-(64/lpr) image
BLK_DECL(blk_one);    // one lane per row on a SELL-64 image
#define BLK_INSTANCE(FN, VT, FT, OT, EPI, NDOT) \
    template unsigned FN<VT, FT, OT, EPI, NDOT>(const BlkCfg &, const DevMat &, const BlkVecs<VT, FT, OT> &);
template <typename VT, typename OT, int NDOT>
unsigned blk_post(const BlkCfg &c, const DevMat &A, bool multi, const PostVecs<VT, OT> &v);

inline unsigned sell_grid(const DevMat &A) { return (unsigned)((A.nslices + SELL_WAVES - 1) / SELL_WAVES); }
// grid of the lanes-per-row kernels (grid-stride over the slices)
inline unsigned blk_grid(const BlkCfg &c, const DevMat &B)
{
    const int64_t wpb = c.threads / 64, g = (B.nslices + wpb - 1) / wpb;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, c.threads == 512 ? 2048 : 4096));
}

// Block matrix pass over the SELL-64 image A or the block image B.
template <typename VT, typename FT, typename OT, int EPI, int NDOT>
unsigned blk_pass(const BlkCfg &c, const DevMat &A, const DevMat &B, const BlkVecs<VT, FT, OT> &v)
{
    if (c.win > 0 && A.nshared > 0 && A.shrun && A.val<VT>()) {
        // stencil image: staged x windows, c.win rows per lane
        if ((c.share & (sizeof(VT) == 8 ? 1 : 2)) && A.wgtab) return blk_wins<VT, FT, OT, EPI, NDOT>(c, A, v);
        return blk_win<VT, FT, OT, EPI, NDOT>(c, A, v);
    }
    if (c.lpr > 1 && B.soff && B.val<VT>()) return blk_rows<VT, FT, OT, EPI, NDOT>(c, B, v);
    return blk_one<VT, FT, OT, EPI, NDOT>(c, A, v);
}

}  // namespace amgk

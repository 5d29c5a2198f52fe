// Device image of one matrix as the launchers hold it (layouts in kernels.h).
#pragma once
#include "kernels.h"

namespace amgk {

// Device arrays of a sliced-ELL (or CSR) image.
struct DevMat {
    int64_t n = 0, ncols = 0, nnz = 0, nslices = 0, stored = 0, nshared = 0;
    double index_bytes = 0.0;
    int idx16 = 1, C = SLICE, sorted = 0;
    int64_t *soff = nullptr, *ibase = nullptr;
    int32_t *col0 = nullptr, *c32 = nullptr, *shoff = nullptr, *perm = nullptr, *shrun = nullptr;
    int32_t *gcol = nullptr;   // split images with 16-bit deltas
    // windows shared by the four slices of a block (batched stencil images)
    int32_t *wgtab = nullptr, *wgst = nullptr;
    int wg_sigma = 0;
    int split = 1;  // wavefronts per slice by the rule (split_waves, or split_waves_blk)
    int one_wave = 0;   // AMG_OPT_SPLIT off
    int xwin = 0;   // single-vector K passes through x windows (shared-offset images with run tables)
    double wg_ratio = 0.0;   // rows the shared windows copy / rows per-wave windows copy
    uint16_t *d16 = nullptr;
    double *v64 = nullptr;
    float *v32 = nullptr;
    // CSR image with `lpr` lanes per row (lpr > 0; FP64, int32 columns) instead
    // of SELL: long or few rows of the smoothed hierarchy
    int lpr = 0;
    int64_t *crp = nullptr;
    int32_t *cci = nullptr;
    double *cv = nullptr;
    bool built() const { return soff || crp; }
    // wavefronts per slice of its passes: the windows are walked by one
    int waves() const { return xwin || one_wave ? 1 : split; }
    template <typename VT> const VT *val() const;
    template <typename IT> const IT *idx() const;
    template <typename VT, typename IT> Sell<VT, IT> sv() const
    {
        return Sell<VT, IT>{n,     ncols, nslices, soff,  ibase, val<VT>(), idx<IT>(), col0,
                            shoff, perm,  shrun,   wgtab, wgst,  xwin, gcol};
    }
};
template <> inline const double *DevMat::val<double>() const { return v64; }
template <> inline const float *DevMat::val<float>() const { return v32; }
template <> inline const uint16_t *DevMat::idx<uint16_t>() const { return d16; }
template <> inline const int32_t *DevMat::idx<int32_t>() const { return c32; }

}  // namespace amgk

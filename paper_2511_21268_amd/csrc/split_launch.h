// Launchers of the passes with several wavefronts per slice (split.h), compiled in a
// translation unit of their own.
#pragma once
#include "blk_launch.h"

namespace amgk {

template <typename VT, typename FT, typename OT, int EPI, int NDOT>
void split_pass(hipStream_t st, const DevMat &A, const BlkVecs<VT, FT, OT> &v, double *partial);
template <typename VT, typename OT, int NDOT>
void split_post(hipStream_t st, const DevMat &A, const PostVecs<VT, OT> &v, double *partial);
template <typename VT>
void split_post_res(hipStream_t st, const DevMat &A, const VT *e, const VT *u, VT *r, const int32_t *agg, const VT *pc,
                    VT *y);
template <int MODE>
void split_cheb(hipStream_t st, const DevMat &A, const double *x, const double *f, double *r, const double *invd,
                double *u, double *dn, double a, double b, int first);

}  // namespace amgk

// Launches of the matrix passes with several wavefronts per slice.
#include "split_launch.h"
#include "split.h"

namespace amgk {

// KER<types..., W> for the image's index type and wavefronts per slice
#define SPLIT_W(KER, IT, ...)                                                                                     \
    do {                                                                                                          \
        if (A.waves() == 4) KER(IT, 4, __VA_ARGS__);                                                                \
        else KER(IT, 8, __VA_ARGS__);                                                                             \
    } while (0)
#define SPLIT(KER, ...)                                \
    do {                                               \
        if (A.idx16) SPLIT_W(KER, uint16_t, __VA_ARGS__); \
        else SPLIT_W(KER, int32_t, __VA_ARGS__);       \
    } while (0)
#define GRID(W) dim3((unsigned)A.nslices), dim3(SLICE * W), 0, st

template <typename VT, typename FT, typename OT, int EPI, int NDOT>
void split_pass(hipStream_t st, const DevMat &A, const BlkVecs<VT, FT, OT> &v, double *partial)
{
#define PASS(IT, W, ...)                                                                                          \
    hipLaunchKernelGGL((k_split<VT, FT, OT, IT, EPI, NDOT, W>), GRID(W), A.sv<VT, IT>(), v.x, v.f, v.invd, v.y,   \
                       v.g0, v.g1, partial, v.coef)
    SPLIT(PASS, );
}

template <typename VT, typename OT, int NDOT>
void split_post(hipStream_t st, const DevMat &A, const PostVecs<VT, OT> &v, double *partial)
{
#define POST(IT, W, ...)                                                                                          \
    hipLaunchKernelGGL((k_split_post<VT, OT, IT, NDOT, W>), GRID(W), A.sv<VT, IT>(), v.e, v.u, v.r, v.invd, v.agg, \
                       v.pc, v.y, v.g0, partial)
    SPLIT(POST, );
}

template <typename VT>
void split_post_res(hipStream_t st, const DevMat &A, const VT *e, const VT *u, VT *r, const int32_t *agg, const VT *pc,
                    VT *y)
{
#define POST_RES(IT, W, ...) \
    hipLaunchKernelGGL((k_split_post_res<VT, IT, W>), GRID(W), A.sv<VT, IT>(), e, u, r, agg, pc, y)
    SPLIT(POST_RES, );
}

template <int MODE>
void split_cheb(hipStream_t st, const DevMat &A, const double *x, const double *f, double *r, const double *invd,
                double *u, double *dn, double a, double b, int first)
{
#define CHEB(IT, W, ...)                                                                                         \
    hipLaunchKernelGGL((k_split_cheb<IT, MODE, W>), GRID(W), A.sv<double, IT>(), x, f, r, invd, u, dn, a, b, first)
    SPLIT(CHEB, );
}

#define INST(VT, FT, OT, EPI, NDOT) \
    template void split_pass<VT, FT, OT, EPI, NDOT>(hipStream_t, const DevMat &, const BlkVecs<VT, FT, OT> &, double *);
BLK_PASSES(INST)
INST(double, double, double, EPI_ADD, 0)
#define INST_POST(VT, OT, NDOT) \
    template void split_post<VT, OT, NDOT>(hipStream_t, const DevMat &, const PostVecs<VT, OT> &, double *);
INST_POST(double, double, 0)
INST_POST(double, double, 1)
INST_POST(float, float, 0)
INST_POST(float, double, 0)
INST_POST(float, double, 1)
template void split_post_res<double>(hipStream_t, const DevMat &, const double *, const double *, double *,
                                     const int32_t *, const double *, double *);
template void split_post_res<float>(hipStream_t, const DevMat &, const float *, const float *, float *,
                                    const int32_t *, const float *, float *);
#define INST_CHEB(MODE)                                                                                          \
    template void split_cheb<MODE>(hipStream_t, const DevMat &, const double *, const double *, double *,        \
                                   const double *, double *, double *, double, double, int);
INST_CHEB(0)
INST_CHEB(1)
INST_CHEB(2)

}  // namespace amgk

// 16-column prolongation fused with the first post-smoothing sweep through K P.
#include "blk_launch.h"
#include "kernels_blk.h"

namespace amgk {

// multi: A is a SELL-(64/lpr) image walked with c.lpr lanes per row, else a
// SELL-64 one with one lane per row (a dot partial per wavefront).
template <typename VT, typename OT, int NDOT>
unsigned blk_post(const BlkCfg &c, const DevMat &A, bool multi, const PostVecs<VT, OT> &v)
{
    if constexpr (NDOT == 0) {
        if (multi && A.waves() > 1) {
#define LAUNCH(IT, LPR)                                                                                           \
    hipLaunchKernelGGL((k_splitb_post<VT, OT, IT, LPR>), dim3((unsigned)A.nslices), dim3(64 * SPLITB_WAVES), 0,   \
                       c.stream, A.sv<VT, IT>(), v.e, v.u, v.r, v.invd, v.agg, v.pc, v.y)
#define LAUNCH_IT(LPR)                   \
    do {                                 \
        if (A.idx16) LAUNCH(uint16_t, LPR); \
        else LAUNCH(int32_t, LPR);       \
    } while (0)
            if (c.lpr == 4) LAUNCH_IT(4);
            else if (c.lpr == 8) LAUNCH_IT(8);
            else LAUNCH_IT(16);
#undef LAUNCH_IT
#undef LAUNCH
            return (unsigned)A.nslices;
        }
    }
    const unsigned g = multi ? blk_grid(c, A) : sell_grid(A);
#define LAUNCH(IT, ...)                                                                                            \
    hipLaunchKernelGGL((__VA_ARGS__), dim3(g), dim3(multi ? c.threads : 256), 0, c.stream, A.sv<VT, IT>(), v.e, v.u, \
                       v.r, v.invd, v.agg, v.pc, v.y, v.g0, (const double *)nullptr, c.partial)
#define LAUNCH_IT(IT)                                                          \
    do {                                                                       \
        if (!multi) LAUNCH(IT, k_sell_blk_post<VT, OT, IT, NDOT>);             \
        else if (c.lpr == 4) LAUNCH(IT, k_sellb_post<VT, OT, IT, NDOT, 4>);    \
        else if (c.lpr == 8) LAUNCH(IT, k_sellb_post<VT, OT, IT, NDOT, 8>);    \
        else LAUNCH(IT, k_sellb_post<VT, OT, IT, NDOT, 16>);                   \
    } while (0)
    if (A.idx16) LAUNCH_IT(uint16_t);
    else LAUNCH_IT(int32_t);
#undef LAUNCH_IT
#undef LAUNCH
    return multi ? g : g * SELL_WAVES;
}
#define INST(VT, OT, NDOT) template unsigned blk_post<VT, OT, NDOT>(const BlkCfg &, const DevMat &, bool, const PostVecs<VT, OT> &);
INST(double, double, 0)
INST(double, double, 1)
INST(float, float, 0)
INST(float, double, 0)
INST(float, double, 1)

}  // namespace amgk

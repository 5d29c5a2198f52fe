// 16-column passes with several lanes per row, and with one.
#include "blk_launch.h"
#include "kernels_blk.h"

namespace amgk {

BLK_DECL(blk_rows)
{
    if constexpr (NDOT == 0) {
        if (A.waves() > 1) {
#define LAUNCH(IT, LPR)                                                                                           \
    hipLaunchKernelGGL((k_splitb<VT, FT, OT, IT, EPI, LPR>), dim3((unsigned)A.nslices), dim3(64 * SPLITB_WAVES), 0, \
                       c.stream, A.sv<VT, IT>(), v.x, v.f, v.invd, v.y, v.coef)
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
    const unsigned g = blk_grid(c, A);
#define LAUNCH(IT, LPR)                                                                                           \
    hipLaunchKernelGGL((k_sellb<VT, FT, OT, IT, EPI, NDOT, LPR>), dim3(g), dim3(c.threads), 0, c.stream,          \
                       A.sv<VT, IT>(), v.x, v.f, v.invd, v.y, v.g0, v.g1, c.partial, v.coef)
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
    return g;
}

BLK_DECL(blk_one)
{
    const unsigned g = sell_grid(A);
#define LAUNCH(IT)                                                                                                \
    hipLaunchKernelGGL((k_sell_blk<VT, FT, OT, IT, EPI, NDOT>), dim3(g), dim3(256), 0, c.stream, A.sv<VT, IT>(), \
                       v.x, v.f, v.invd, v.y, v.g0, v.g1, c.partial, v.coef)
    if (A.idx16) LAUNCH(uint16_t);
    else LAUNCH(int32_t);
#undef LAUNCH
    return g * SELL_WAVES;   // dot partials: one per wavefront
}

#define INST(...) BLK_INSTANCE(blk_rows, __VA_ARGS__) BLK_INSTANCE(blk_one, __VA_ARGS__)
BLK_PASSES(INST)

}  // namespace amgk

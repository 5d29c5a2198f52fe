// 16-column stencil passes from LDS windows of X: windows per wave.
#include "blk_launch.h"
#include "kernels_blk.h"

namespace amgk {

// The grid is padded to a multiple of the XCD count (XCD-aware slice order);
// dot partials: one per wavefront of a logical block.
BLK_DECL(blk_win)
{
    const dim3 grid(xcd_grid(sell_grid(A)));
#define LAUNCH(IT, R)                                                                                            \
    hipLaunchKernelGGL((k_sellw_blk<VT, FT, OT, IT, EPI, NDOT, R>), grid, dim3(256), 0, c.stream, A.sv<VT, IT>(), v.x, \
                       v.f, v.invd, v.y, v.g0, v.g1, c.partial, v.coef)
    if (A.idx16) {
        if (c.win == 2) LAUNCH(uint16_t, 2);
        else LAUNCH(uint16_t, 4);
    } else {
        if (c.win == 2) LAUNCH(int32_t, 2);
        else LAUNCH(int32_t, 4);
    }
#undef LAUNCH
    return sell_grid(A) * SELL_WAVES;
}
#define INST(...) BLK_INSTANCE(blk_win, __VA_ARGS__)
BLK_PASSES(INST)

}  // namespace amgk

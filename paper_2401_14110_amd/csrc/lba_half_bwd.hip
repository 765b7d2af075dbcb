// lba_half_bwd.hip -- instantiations of the recompute call on packed FP16 carriers (lba_half_bwd.h).
#include "lba_half_bwd.h"
#include "lba_launch.h"

namespace lba {

template <int PM, bool UF, int AMODE>
static hipError_t launch_one(const Plan& pl, hipStream_t st) {
    const dim3 block(256);
    if (pl.mix_tail > 0) {                                     // sequential order
        if (pl.order != LBA_ORDER_SEQ || pl.kp.mix_half != 0 || pl.kp.mix_tail16 != 0) return hipErrorInvalidValue;
        hipLaunchKernelGGL((lba_half_bwd_mixed_kernel<PM, UF, AMODE>), dim3(pl.grid_x, 1, 1), block, 0, st, pl.kp);
    } else if (pl.order == LBA_ORDER_SEQ) {
        hipLaunchKernelGGL((lba_half_bwd_kernel<PM, LBA_ORDER_SEQ, UF, AMODE>), dim3(pl.grid_x, pl.grid_y, 1), block, 0, st, pl.kp);
    } else {
        // the planner asks for truncated products and for im2col rows under the sequential order only
        if constexpr (PM == PM_FLUSH && AMODE == 0)
            hipLaunchKernelGGL((lba_half_bwd_kernel<PM, LBA_ORDER_CHUNK16, UF, AMODE>), dim3(pl.grid_x, pl.grid_y, 1), block, 0, st, pl.kp);
        else
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int PM>
static hipError_t launch_product(const Plan& pl, hipStream_t st) {
    const bool uf = pl.kp.uf_mask != nullptr || pl.kp.uf_mask2 != nullptr;
    if (pl.kp.conv) return uf ? launch_one<PM, true, 2>(pl, st) : launch_one<PM, false, 2>(pl, st);
    return uf ? launch_one<PM, true, 0>(pl, st) : launch_one<PM, false, 0>(pl, st);
}

hipError_t launch_half_bwd(const Plan& pl, hipStream_t st) {
    if (pl.events != 1 || pl.round != LBA_ROUND_FLOOR || pl.kp.batch != 1 || pl.tm != 4 || pl.tn != 4) return hipErrorInvalidValue;
    if (pl.prod_mode == PM_FLUSH) return launch_product<PM_FLUSH>(pl, st);
    if (pl.prod_mode == PM_TRUNC) return launch_product<PM_TRUNC>(pl, st);
    return hipErrorInvalidValue;
}

}  // namespace lba

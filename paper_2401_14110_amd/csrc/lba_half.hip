// lba_half.hip -- instantiations of the forward kernels on packed FP16 carriers (lba_rows.h) for row-major matrices.
#include "lba_rows.h"
#include "lba_launch.h"

namespace lba {

// (truncated products come on the 4 x 4 lane block and mixed grids only; the 2 x 2 block has waves that stage)
template <int PM, int ORDER, int AMODE>
static hipError_t launch_one(const Plan& pl, hipStream_t st) {
    const dim3 grid(pl.grid_x, pl.grid_y, pl.kp.batch), block(256);
    if (pl.mix_tail > 0) {
        hipLaunchKernelGGL((lba_half_mixed_kernel<PM, ORDER, AMODE>), grid, block, 0, st, pl.kp);
        return hipGetLastError();
    }
    if (pl.tm == 4 && pl.tn == 4) {
        hipLaunchKernelGGL((lba_half_kernel<4, 4, PM, ORDER, AMODE>), grid, block, 0, st, pl.kp);
        return hipGetLastError();
    }
    if constexpr (PM != PM_TRUNC) {
        if (pl.tm == 2 && pl.tn == 4) {
            hipLaunchKernelGGL((lba_half_kernel<2, 4, PM, ORDER, AMODE>), grid, block, 0, st, pl.kp);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidValue;
}

template <int ORDER, int AMODE>
static hipError_t launch_order(const Plan& pl, hipStream_t st) {
    if (pl.prod_mode == PM_IDENT) return launch_one<PM_IDENT, ORDER, AMODE>(pl, st);
    if (pl.prod_mode == PM_FLUSH) return launch_one<PM_FLUSH, ORDER, AMODE>(pl, st);
    if (pl.prod_mode == PM_TRUNC) return launch_one<PM_TRUNC, ORDER, AMODE>(pl, st);
    return hipErrorInvalidValue;
}

template <int PM, int ORDER>
static hipError_t launch_staged(const Plan& pl, hipStream_t st) {
    const dim3 grid(pl.grid_x, pl.grid_y, pl.kp.batch), block(512);
    if (pl.mix_tail > 0)              hipLaunchKernelGGL((lba_half_staged_kernel<2, PM, ORDER>), grid, block, 0, st, pl.kp);
    else if constexpr (PM != PM_TRUNC) hipLaunchKernelGGL((lba_half_staged_kernel<4, PM, ORDER>), grid, block, 0, st, pl.kp);
    else                              return hipErrorInvalidValue;   // (the 2 x 2 lane block has no truncated products: pick_tile)
    return hipGetLastError();
}
template <int ORDER>
static hipError_t launch_staged(const Plan& pl, hipStream_t st) {
    if (pl.prod_mode == PM_IDENT) return launch_staged<PM_IDENT, ORDER>(pl, st);
    if (pl.prod_mode == PM_FLUSH) return launch_staged<PM_FLUSH, ORDER>(pl, st);
    if (pl.prod_mode == PM_TRUNC) return launch_staged<PM_TRUNC, ORDER>(pl, st);
    return hipErrorInvalidValue;
}

hipError_t launch_half(const Plan& pl, hipStream_t st) {
    if (pl.events || pl.round != LBA_ROUND_FLOOR || pl.kp.conv || !pl.kp.h_on) return hipErrorInvalidValue;
    if (pl.staged) {                                           // 32 x 16 tiles throughout, or 32 x 32
        if (pl.mix_tail > 0 ? !pl.kp.mix_tail16 || pl.kp.mix_main + pl.kp.mix_half != 0 : pl.tm != 2 || pl.tn != 2) return hipErrorInvalidValue;
        return pl.order == LBA_ORDER_CHUNK16 ? launch_staged<LBA_ORDER_CHUNK16>(pl, st) : launch_staged<LBA_ORDER_SEQ>(pl, st);
    }
    if (pl.kp.ld_align == 16)
        return pl.order == LBA_ORDER_CHUNK16 ? launch_order<LBA_ORDER_CHUNK16, 0>(pl, st) : launch_order<LBA_ORDER_SEQ, 0>(pl, st);
    return pl.order == LBA_ORDER_CHUNK16 ? launch_order<LBA_ORDER_CHUNK16, 3>(pl, st) : launch_order<LBA_ORDER_SEQ, 3>(pl, st);
}

}  // namespace lba

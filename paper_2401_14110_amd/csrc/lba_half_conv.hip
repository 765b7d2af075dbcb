// lba_half_conv.hip -- instantiations of the forward kernels on packed FP16 carriers (lba_rows.h) for im2col rows of an NHWC tensor.
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

template <int PM, int CONV, int ORDER>
static hipError_t launch_staged(const Plan& pl, hipStream_t st) {
    const dim3 grid(pl.grid_x, pl.grid_y, pl.kp.batch), block(512);
    if (pl.mix_tail > 0) hipLaunchKernelGGL((lba_half_staged_conv_kernel<2, PM, CONV, ORDER>), grid, block, 0, st, pl.kp);
    else                 hipLaunchKernelGGL((lba_half_staged_conv_kernel<4, PM, CONV, ORDER>), grid, block, 0, st, pl.kp);
    return hipGetLastError();
}
template <int CONV, int ORDER>
static hipError_t launch_staged(const Plan& pl, hipStream_t st) {
    return pl.prod_mode == PM_IDENT ? launch_staged<PM_IDENT, CONV, ORDER>(pl, st) : pl.prod_mode == PM_FLUSH ? launch_staged<PM_FLUSH, CONV, ORDER>(pl, st) : hipErrorInvalidValue;
}

hipError_t launch_half_conv(const Plan& pl, hipStream_t st) {
    if (pl.events || pl.round != LBA_ROUND_FLOOR || !pl.kp.conv || !pl.kp.h_on) return hipErrorInvalidValue;
    if (pl.staged) {                                           // 32 x 16 tiles throughout, or 32 x 32
        if (pl.mix_tail > 0 ? !pl.kp.mix_tail16 || pl.kp.mix_main + pl.kp.mix_half != 0 : pl.tm != 2 || pl.tn != 2) return hipErrorInvalidValue;
        if (pl.order == LBA_ORDER_CHUNK16) return pl.kp.cv_vec ? launch_staged<1, LBA_ORDER_CHUNK16>(pl, st) : launch_staged<2, LBA_ORDER_CHUNK16>(pl, st);
        return pl.kp.cv_vec ? launch_staged<1, LBA_ORDER_SEQ>(pl, st) : launch_staged<2, LBA_ORDER_SEQ>(pl, st);
    }
    if (pl.kp.cv_vec && pl.kp.ld_align == 16)
        return pl.order == LBA_ORDER_CHUNK16 ? launch_order<LBA_ORDER_CHUNK16, 2>(pl, st) : launch_order<LBA_ORDER_SEQ, 2>(pl, st);
    return pl.order == LBA_ORDER_CHUNK16 ? launch_order<LBA_ORDER_CHUNK16, 4>(pl, st) : launch_order<LBA_ORDER_SEQ, 4>(pl, st);
}

}  // namespace lba

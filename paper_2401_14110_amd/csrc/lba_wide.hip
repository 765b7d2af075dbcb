// lba_wide.hip -- instantiations of the forward kernels on packed FP16 carriers (lba_rows.h) whose accumulator reaches beyond FP16's range.
#include "lba_rows.h"
#include "lba_launch.h"

namespace lba {

template <int ORDER, int AMODE, int RANGE>
static hipError_t launch_one(const Plan& pl, hipStream_t st) {
    const dim3 grid(pl.grid_x, pl.grid_y, pl.kp.batch), block(256);
    if (pl.mix_tail > 0)                    hipLaunchKernelGGL((lba_wide_mixed_kernel<ORDER, AMODE, RANGE>), grid, block, 0, st, pl.kp);
    else if (pl.tm == 4 && pl.tn == 4)      hipLaunchKernelGGL((lba_wide_kernel<4, 4, ORDER, AMODE, RANGE>), grid, block, 0, st, pl.kp);
    else if (pl.tm == 2 && pl.tn == 4)      hipLaunchKernelGGL((lba_wide_kernel<2, 4, ORDER, AMODE, RANGE>), grid, block, 0, st, pl.kp);
    else if (pl.tm == 2 && pl.tn == 2)      hipLaunchKernelGGL((lba_wide_kernel<2, 2, ORDER, AMODE, RANGE>), grid, block, 0, st, pl.kp);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int ORDER, int AMODE>
static hipError_t launch_range(const Plan& pl, hipStream_t st) {
    return pl.kp.h_range == 2 ? launch_one<ORDER, AMODE, 2>(pl, st) : launch_one<ORDER, AMODE, 1>(pl, st);
}

template <int AMODE>
static hipError_t launch_order(const Plan& pl, hipStream_t st) {
    return pl.order == LBA_ORDER_CHUNK16 ? launch_range<LBA_ORDER_CHUNK16, AMODE>(pl, st) : launch_range<LBA_ORDER_SEQ, AMODE>(pl, st);
}

#if LBA_WIDE_CONV
hipError_t launch_wide_conv(const Plan& pl, hipStream_t st) {
    if (pl.events || pl.round != LBA_ROUND_FLOOR || !pl.kp.conv || !pl.kp.h_on || !pl.kp.h_range || pl.prod_mode != PM_FLUSH) return hipErrorInvalidValue;
    return pl.kp.cv_vec && pl.kp.ld_align == 16 ? launch_order<2>(pl, st) : launch_order<4>(pl, st);
}
#else
hipError_t launch_wide(const Plan& pl, hipStream_t st) {
    if (pl.events || pl.round != LBA_ROUND_FLOOR || pl.kp.conv || !pl.kp.h_on || !pl.kp.h_range || pl.prod_mode != PM_FLUSH) return hipErrorInvalidValue;
    return pl.kp.ld_align == 16 ? launch_order<0>(pl, st) : launch_order<3>(pl, st);
}
#endif

}  // namespace lba

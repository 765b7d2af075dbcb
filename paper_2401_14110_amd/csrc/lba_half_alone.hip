// lba_half_alone.hip -- kernels on packed FP16 carriers for launches whose large workgroups number at most one per CU, so that a wave has its
// SIMD to itself.
//
// What bounds them: one wave's issue.  It has nobody to take turns with (a change of priority is an instruction like any other, two a step),
// a list of non-zero codes costs it the latency of a read per step, which no other wave hides, and registers are there for the
// taking: operands are read four pairs of steps ahead and a step's products stand before the mask of the step ahead.  Kernels of their own,
// because both forms in one kernel cost the other one 3 % (its reads were moved before the branch).
// Measured (us), lane blocks before there were rows / rows with turns and lists / here, 16384 x 64 x 1024 (256 workgroups):
//   overflow plane  75 / 83, behind a ReLU 89 / 73      in chunks  79 /  83 /  75      both planes 203 / 212 / 202
//   truncated products, forward  77 / 85, behind a ReLU 87 / 77
// and 18920 x 24 x 6272, 256 workgroups of 48 x 64 before 208 of 32 x 32: 347 / 377 / 331 (the small ones are done first; with 256 or more of
// them, two and more waves on every SIMD, turns are the faster: 19200 x 64 x 1024 74 / 69, 73 without).
#include "lba_rows.h"
#include "lba_launch.h"

namespace lba {

// The recompute call on at most 256 workgroups of 64 x 64.  T 2: workgroups of 32 x 32, a CU's share of which is the smaller the fewer
// there are, and whose chains are a fourth of a wave's work.  T 4: 64 x 64, for the overflow plane under the sequential order on more than 192
// of them, where a wave alone on its SIMD issues as much as the four of the small ones (900 x 900 x 700, training step, 151 us, 152), and for
// widths that are no multiple of 32, whose small tiles write parts of cache lines (partial_lines, lba_plan.cpp; 64 x 64 and 32 x 32, 256 workgroups, both planes,
// N = 190, K = 1000 1.24 times as long, 193 to 256, K = 513 to 768 0.88 to 1.09, mean 0.95, to 2500 0.93 to 1.24, in chunks from 513 0.97 to 1.19, K = 300 0.84 to 1.09, 192 workgroups 0.68 to 0.93; the overflow plane in chunks,
// N = 159, K = 1501 124.6 and 192 us, 200 to 224 workgroups, K > 1024, 1.04 to 1.35 times as long, K = 300, 256 workgroups 31.5 and 34.7; 161 to 192, K > 1024, in
// either order 0.77 to 1.00).
// 64 x 64 -> 32 x 32, both planes: 500 x 500 x 700 143 -> 60 us, 700 x 700 145 -> 78, 1024 x 1024 142 -> 122; training steps, K = 700:
// 500 x 500 115 -> 84, 700 x 700 125 -> 103, 1024 x 700 145 -> 133, in chunks 149 -> 108, 179 -> 131, 194 -> 180, 1024 x 1024 210 -> 207.
template <int T, int PM, int ORDER, bool UF, int AMODE>
__global__ void __launch_bounds__(256, UF ? (ORDER == LBA_ORDER_CHUNK16 ? 2 : 3) : (T == 4 ? 1 : 2)) lba_half_bwd_alone_kernel(const KParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[UF ? 2 * HalfTile<T, T, 16>::STAGE : RowTile<4 * T, 2 * T>::WORDS];
    if constexpr (UF) half_bwd_body<T, T, PM, ORDER, AMODE, false>(p, smem, blockIdx.x * 16 * T, blockIdx.y * 16 * T);
    else              rows_body<4 * T, 2 * T, PM, ORDER, AMODE, 0, true, true>(p, smem, blockIdx.x * 16 * T, blockIdx.y * 16 * T);
}
template <int PM, int ORDER, int AMODE>
__global__ void __launch_bounds__(256, 1) lba_half_alone_kernel(const KParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[RowTile<16, 8>::WORDS];
    rows_body<16, 8, PM, ORDER, AMODE, 0, false, true>(p, smem, blockIdx.x * 64, blockIdx.y * 64);
}
template <int PM, int ORDER, int AMODE>
__global__ void __launch_bounds__(256, 2) lba_half_alone_mixed_kernel(const KParams p) { rows_mixed<PM, ORDER, AMODE, 0, true>(p); }

template <int PM, int ORDER, bool UF, int AMODE>
static hipError_t launch_bwd(const Plan& pl, hipStream_t st) {
    const dim3 grid(pl.grid_x, pl.grid_y, 1), block(256);
    if (pl.tm == 2) hipLaunchKernelGGL((lba_half_bwd_alone_kernel<2, PM, ORDER, UF, AMODE>), grid, block, 0, st, pl.kp);
    else            hipLaunchKernelGGL((lba_half_bwd_alone_kernel<4, PM, ORDER, UF, AMODE>), grid, block, 0, st, pl.kp);
    return hipGetLastError();
}
template <int PM, int ORDER>
static hipError_t launch_bwd(const Plan& pl, hipStream_t st) {
    const bool uf = pl.kp.uf_mask != nullptr || pl.kp.uf_mask2 != nullptr, aligned = pl.kp.ld_align == 16;
    if constexpr (ORDER == LBA_ORDER_SEQ) {                    // im2col rows come under the sequential order only
        if (pl.kp.conv)
            return uf ? launch_bwd<PM, ORDER, true, 2>(pl, st) : aligned && pl.kp.cv_vec ? launch_bwd<PM, ORDER, false, 2>(pl, st) : launch_bwd<PM, ORDER, false, 4>(pl, st);
    } else if (pl.kp.conv) {
        return hipErrorInvalidValue;
    }
    if (uf) return pl.kp.N % 4 ? launch_bwd<PM, ORDER, true, 3>(pl, st) : launch_bwd<PM, ORDER, true, 0>(pl, st);
    return aligned ? launch_bwd<PM, ORDER, false, 0>(pl, st) : launch_bwd<PM, ORDER, false, 3>(pl, st);
}
// truncated products under the sequential order only (lba_half_bwd.hip)
hipError_t launch_half_bwd_alone(const Plan& pl, hipStream_t st) {
    if (pl.events != 1 || pl.mix_tail != 0 || pl.tm != pl.tn || (pl.tm != 2 && pl.tm != 4)) return hipErrorInvalidValue;
    if (pl.prod_mode == PM_TRUNC) return pl.order == LBA_ORDER_SEQ ? launch_bwd<PM_TRUNC, LBA_ORDER_SEQ>(pl, st) : hipErrorInvalidValue;
    if (pl.prod_mode != PM_FLUSH) return hipErrorInvalidValue;
    return pl.order == LBA_ORDER_SEQ ? launch_bwd<PM_FLUSH, LBA_ORDER_SEQ>(pl, st) : launch_bwd<PM_FLUSH, LBA_ORDER_CHUNK16>(pl, st);
}

template <int ORDER, int AMODE>
static hipError_t launch_one(const Plan& pl, hipStream_t st) {
    const dim3 grid(pl.grid_x, pl.grid_y, pl.kp.batch), block(256);
    if (pl.mix_tail > 0) {
        if (pl.prod_mode != PM_FLUSH) return hipErrorInvalidValue;
        hipLaunchKernelGGL((lba_half_alone_mixed_kernel<PM_FLUSH, ORDER, AMODE>), grid, block, 0, st, pl.kp);
    } else {
        if constexpr (AMODE == 0 || AMODE == 3) {
            if (pl.prod_mode != PM_TRUNC || pl.tm != 4 || pl.tn != 4) return hipErrorInvalidValue;
            hipLaunchKernelGGL((lba_half_alone_kernel<PM_TRUNC, ORDER, AMODE>), grid, block, 0, st, pl.kp);
        } else {
            return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}
template <int AMODE>
static hipError_t launch_order(const Plan& pl, hipStream_t st) {
    return pl.order == LBA_ORDER_CHUNK16 ? launch_one<LBA_ORDER_CHUNK16, AMODE>(pl, st) : launch_one<LBA_ORDER_SEQ, AMODE>(pl, st);
}
hipError_t launch_half_alone(const Plan& pl, hipStream_t st) {
    if (pl.kp.conv) return pl.kp.cv_vec && pl.kp.ld_align == 16 ? launch_order<2>(pl, st) : launch_order<4>(pl, st);
    return pl.kp.ld_align == 16 ? launch_order<0>(pl, st) : launch_order<3>(pl, st);
}

}  // namespace lba

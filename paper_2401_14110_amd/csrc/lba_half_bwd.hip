// lba_half_bwd.hip -- instantiations of the recompute call on packed FP16 carriers (lba_half_bwd.h).
#include "lba_rows.h"
#include "lba_launch.h"

namespace lba {

// The grids of lba_fast_bwd_kernel and lba_fast_bwd_mixed_kernel.  With an underflow plane AMODE 0: a row-major matrix of any code format
// with E <= 4, 2: im2col rows of an NHWC tensor, 3: as 0, N no multiple of 4; without one as lba_half_kernel.
// Chunks without an underflow plane: at four waves per SIMD 33 registers are spilled, which 819 workgroups and more hide (3985 x 770 x 771,
// training step 648 us against 662 at three, 630 with a tail) and 257 to 768 do not (24576 x 64 x 1024 114 against 109).
template <int PM, int ORDER, bool UF, int AMODE>
__global__ void __launch_bounds__(256, ORDER == LBA_ORDER_CHUNK16 && UF ? 2 : UF || ORDER == LBA_ORDER_CHUNK16 ? 3 : 4) lba_half_bwd_kernel(const KParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[UF ? 2 * HalfTile<4, 4, 16>::STAGE : RowTile<16, 8>::WORDS];
    if constexpr (UF) half_bwd_body<4, 4, PM, ORDER, AMODE>(p, smem, blockIdx.x * 64, blockIdx.y * 64);
    else              rows_body<16, 8, PM, ORDER, AMODE, 0, true>(p, smem, blockIdx.x * 64, blockIdx.y * 64);
}

template <int PM, int ORDER, bool UF, int AMODE>
__global__ void __launch_bounds__(256, UF || ORDER == LBA_ORDER_CHUNK16 ? 3 : 4) lba_half_bwd_mixed_kernel(const KParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[UF ? 2 * HalfTile<4, 4, 16>::STAGE : RowTile<16, 8>::WORDS];
    const int b = blockIdx.x;
    if (b < p.mix_main) {                                      // uniform
        const int by = b / p.mix_gx_main, bx = b - by * p.mix_gx_main;
        if constexpr (UF) half_bwd_body<4, 4, PM, ORDER, AMODE>(p, smem, bx * 64, by * 64);
        else              rows_body<16, 8, PM, ORDER, AMODE, 0, true>(p, smem, bx * 64, by * 64);
    } else {
        const int t = b - p.mix_main;
        const int by = t / p.mix_gx_tail, bx = t - by * p.mix_gx_tail;
        if constexpr (UF) half_bwd_body<2, 2, PM, ORDER, AMODE>(p, smem, p.mix_m_main + bx * 32, by * 32);
        else              rows_body<8, 4, PM, ORDER, AMODE, 0, true>(p, smem, p.mix_m_main + bx * 32, by * 32);
    }
}

template <int PM, bool UF, int AMODE>
static hipError_t launch_one(const Plan& pl, hipStream_t st) {
    const dim3 block(256);
    if (pl.mix_tail > 0 && (pl.kp.mix_half != 0 || pl.kp.mix_tail16 != 0)) return hipErrorInvalidValue;
    if (pl.mix_tail > 0 && pl.order == LBA_ORDER_SEQ) {
        hipLaunchKernelGGL((lba_half_bwd_mixed_kernel<PM, LBA_ORDER_SEQ, UF, AMODE>), dim3(pl.grid_x, 1, 1), block, 0, st, pl.kp);
    } else if (pl.mix_tail > 0) {                              // chunks: the overflow planes alone
        if constexpr (PM == PM_FLUSH && !UF && (AMODE == 0 || AMODE == 3))
            hipLaunchKernelGGL((lba_half_bwd_mixed_kernel<PM, LBA_ORDER_CHUNK16, UF, AMODE>), dim3(pl.grid_x, 1, 1), block, 0, st, pl.kp);
        else
            return hipErrorInvalidValue;
    } else if (pl.order == LBA_ORDER_SEQ) {
        hipLaunchKernelGGL((lba_half_bwd_kernel<PM, LBA_ORDER_SEQ, UF, AMODE>), dim3(pl.grid_x, pl.grid_y, 1), block, 0, st, pl.kp);
    } else {
        // the planner asks for truncated products and for im2col rows under the sequential order only
        if constexpr (PM == PM_FLUSH && (AMODE == 0 || AMODE == 3))
            hipLaunchKernelGGL((lba_half_bwd_kernel<PM, LBA_ORDER_CHUNK16, UF, AMODE>), dim3(pl.grid_x, pl.grid_y, 1), block, 0, st, pl.kp);
        else
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int PM>
static hipError_t launch_product(const Plan& pl, hipStream_t st) {
    const bool uf = pl.kp.uf_mask != nullptr || pl.kp.uf_mask2 != nullptr;
    const bool aligned = pl.kp.ld_align == 16;
    if (pl.kp.conv) return uf ? launch_one<PM, true, 2>(pl, st) : aligned && pl.kp.cv_vec ? launch_one<PM, false, 2>(pl, st) : launch_one<PM, false, 4>(pl, st);
    return uf ? (pl.kp.N % 4 ? launch_one<PM, true, 3>(pl, st) : launch_one<PM, true, 0>(pl, st)) : aligned ? launch_one<PM, false, 0>(pl, st) : launch_one<PM, false, 3>(pl, st);
}

hipError_t launch_half_bwd(const Plan& pl, hipStream_t st) {
    if (pl.events != 1 || pl.round != LBA_ROUND_FLOOR || pl.kp.batch != 1 || pl.tm != 4 || pl.tn != 4) return hipErrorInvalidValue;
    if (pl.prod_mode == PM_FLUSH) return launch_product<PM_FLUSH>(pl, st);
    if (pl.prod_mode == PM_TRUNC) return launch_product<PM_TRUNC>(pl, st);
    return hipErrorInvalidValue;
}

}  // namespace lba

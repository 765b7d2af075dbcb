// lba_half.h -- the forward tile of lba_device.h on packed FP16 carriers: two chains per register.
//
// A chain whose accumulator has at most 11 significant bits and 29 binades (the 12-bit M7E4 and the whole E <= 4 row
// of the format sweep) fits an FP16 number, and under floor rounding every step is exact on it:
//   * the domain puts R_UF of Q_acc at 2^-14, FP16's smallest normal, with FP16 results below it flushed (and
//     denormal inputs read: MODE[7:6] = 1), so the flush of the multiply-add is Q_acc's underflow, as in the FP32 tile;
//   * v_pk_fma_f16 forms p * kc + S exactly and rounds it once, toward zero (MODE[3:2] = 3), to 11 bits; truncating 11
//     and then M + 1 <= 11 bits equals truncating the exact sum to M + 1 bits;
//   * a product of at most 11 bits is exact; its domain has R_UF of Q_prod at 2^-14, so the multiply's flush is
//     Q_prod's, and the planner admits the format only if the largest product stays below FP16's largest number;
//   * a sum beyond FP16's range ends at +-65504 (or infinity), which is clamped to R_OF like every sum beyond R_OF.
// No bit differs from the FP32 tile or from the definition: FP16 is the narrower register that the caller's own
// accumulator format fits, not a reduced precision.
//
// What bounds it: VALU issue.  The FP32 step of a chain is mul, fma, and at one wave64 instruction per 2.3 to 2.8 cycles
// with several waves per SIMD (6.8 cycles per chain in the issue-rate probe, 12.9 with one wave); the packed step of two
// chains is v_pk_mul, v_pk_fma (4.3 cycles each, whatever the number of waves) and one v_and (6.1 per chain, 7.5 with
// one wave).  It also reads a quarter of the LDS bytes per step, and 64 steps take the LDS of 32: with stages of 32 steps
// every shape measured 3-8 % slower, with 5 to 8 waves per SIMD instead of 4 none faster.  The forward call's tile is lba_rows.h;
// the 4 x 4 lane block here serves the recompute call (lba_half_bwd.h).

#ifndef LBA_HALF_H_
#define LBA_HALF_H_

#include "lba_device.h"
#include "lba_piece.h"

namespace lba {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void set_round_zero_f16()  { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3\n\ts_nop 1" ::: "memory"); }
// FP16: denormal inputs are read, denormal results flushed
__device__ __forceinline__ void set_flush_out_f16()   { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 6, 2), 1\n\ts_nop 1" ::: "memory"); }

template <int N> struct IntConst { static constexpr int value = N; };

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ uint32_t as_u32(h2 h) { return __builtin_bit_cast(uint32_t, h); }
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
// the largest of the wave's values in both halves of a word, in lane 63
__device__ __forceinline__ uint32_t wave_max_u16(uint32_t m) {
    const auto step = [&](auto ctrl) { m = pk_max_u16(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, decltype(ctrl)::value, 0xF, 0xF, true)); };
    step(IntConst<0xB1>{});                                    // lane ^ 1, lane ^ 2, the other half of 8 and of 16
    step(IntConst<0x4E>{});
    step(IntConst<0x141>{});
    step(IntConst<0x140>{});
    m = pk_max_u16(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x142, 0xA, 0xF, false));   // row 0 to 1, 2 to 3
    m = pk_max_u16(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x143, 0xC, 0xF, false));   // row 1 to 2 and 3
    return m;
}
// the larger half of a word of two non-negative FP16 numbers, as a float
__device__ __forceinline__ float max_half(uint32_t m) {
    const uint16_t lo = (uint16_t)m, hi = (uint16_t)(m >> 16);
    return (float)__builtin_bit_cast(_Float16, lo > hi ? lo : hi);
}

// Per-wave constants, forced into vector registers (see FastConst).
struct HalfConst {
    h2 kc, rof, nrof;
    uint32_t mask, maskp;
};

// Geometry of one workgroup tile: LX lanes along n, 256 / LX along m, TM x TN outputs per lane (TN even: the pairs are
// neighbours along n).  A k-tile in LDS is HBK (64) steps deep: A as words (k, k + 1) of one row, [k / 2][row], so that one
// read serves two steps (the step's half is picked by the instruction); B as words (n, n + 1) of one k, [k][n / 2].
template <int TM, int TN, int LX>
struct HalfTile {
    static constexpr int BM = 256 / LX * TM, BN = LX * TN;
    static constexpr int BMP = Stage<BM, HBK>::kPitch;                     // words per k pair of A
    static constexpr int BNP = BN / 2;                                     // words per k of B
    static constexpr int A_WORDS = HBK / 2 * BMP, STAGE = A_WORDS + HBK * BNP;
};

// Decodes the 16 codes of a piece into FP16: a code's magnitude bits are the exponent and mantissa of an FP16 number
// (value * 2^(bias - 15), subnormals included; every code of a format with E <= 4 is finite there, so E4M3's two NaN codes
// come out as +-480), then one exact multiply by a power of two.  w[j] holds the codes 2j, 2j + 1.
__device__ __forceinline__ void decode_half(const uint4& v, int shift, uint32_t keep, uint32_t scale, uint32_t (&w)[8]) {
    const uint32_t q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t lo = __builtin_amdgcn_perm(q[i], q[i], 0x010C000Cu), hi = __builtin_amdgcn_perm(q[i], q[i], 0x030C020Cu);
        w[2 * i + 0] = __builtin_bit_cast(uint32_t, (i16x2)(__builtin_bit_cast(i16x2, lo) >> (int16_t)shift)) & keep;
        w[2 * i + 1] = __builtin_bit_cast(uint32_t, (i16x2)(__builtin_bit_cast(i16x2, hi) >> (int16_t)shift)) & keep;
    }
    if (scale != 0x3C003C00u) {                                // uniform; a scaled operand may be an FP16 denormal number
        asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 6, 2), 3\n\t"
                     "s_nop 1\n\t"
                     "v_pk_mul_f16 %0, %0, %8\n\tv_pk_mul_f16 %1, %1, %8\n\tv_pk_mul_f16 %2, %2, %8\n\tv_pk_mul_f16 %3, %3, %8\n\t"
                     "v_pk_mul_f16 %4, %4, %8\n\tv_pk_mul_f16 %5, %5, %8\n\tv_pk_mul_f16 %6, %6, %8\n\tv_pk_mul_f16 %7, %7, %8\n\t"
                     "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 6, 2), 1\n\t"
                     "s_nop 1"
                     : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), "+v"(w[7])
                     : "v"(scale));
    }
}

// Sum of the squares of a piece's 16 values, from above: the constant covers 16 denormal values, should the dot product
// flush them.
__device__ __forceinline__ float piece_norm2(const uint32_t (&w)[8]) {
    float n = 0x1p-24f;
#pragma unroll
    for (int j = 0; j < 8; ++j) n = __builtin_amdgcn_fdot2(as_h2(w[j]), as_h2(w[j]), n, false);
    return n;
}

template <int ROWS>
__device__ __forceinline__ void store_half_a(uint32_t* __restrict__ dst, int tid, const uint32_t (&w)[8]) {
    if (tid < Stage<ROWS, HBK>::kChunks) {
        const int row = Stage<ROWS, HBK>::slot(tid % ROWS), kq = tid / ROWS;
#pragma unroll
        for (int j = 0; j < 8; ++j) dst[(kq * 8 + j) * Stage<ROWS, HBK>::kPitch + row] = w[j];
    }
}

// B's words pair neighbouring columns: lanes 2i and 2i + 1 hold columns n and n + 1, exchange their words and keep the
// even / the odd k of every pair.  (Whole waves take part or none: a tile has a multiple of 64 pieces.)
template <int COLS>
__device__ __forceinline__ void store_half_b(uint32_t* __restrict__ dst, int tidb, const uint32_t (&w)[8]) {
    static_assert(Stage<COLS, HBK>::kChunks % 64 == 0 && COLS % 2 == 0, "neighbouring columns in neighbouring lanes");
    if (tidb >= 0 && tidb < Stage<COLS, HBK>::kChunks) {
        const int col = tidb % COLS, kq = tidb / COLS;
        const uint32_t sel = (col & 1) ? 0x03020706u : 0x05040100u;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[j], 0xB1, 0xF, 0xF, true);   // the neighbour's word
            dst[(kq * 16 + 2 * j + (col & 1)) * (COLS / 2) + (col >> 1)] = __builtin_amdgcn_perm(other, w[j], sel);
        }
    }
}

// A step's products (PM_IDENT: none).  HI: the step is the odd k of its pair of steps.
template <int PM, bool HI, int TM, int TN, bool PRIO = (TM * TN > 4)>
__device__ __forceinline__ void half_products(h2 (&q)[TM][TN / 2], const uint32_t (&a)[TM], const uint32_t (&b)[TN / 2], const HalfConst& c) {
    if (PM != PM_IDENT) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const h2 w = as_h2(a[i]);
            const h2 ab = HI ? __builtin_shufflevector(w, w, 1, 1) : __builtin_shufflevector(w, w, 0, 0);
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) q[i][j] = ab * as_h2(b[j]);   // exact; flushed below Q_prod's R_UF
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if (PM == PM_TRUNC) {
        issue_last<PRIO>();
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) q[i][j] = as_h2(as_u32(q[i][j]) & c.maskp);
        __builtin_amdgcn_sched_barrier(0);
        issue_first<PRIO>();
    }
}

// The sums of a step: one rounding of the exact sum toward zero.
template <int PM, bool HI, int TM, int TN>
__device__ __forceinline__ void half_sums(h2 (&acc)[TM][TN / 2], const h2 (&q)[TM][TN / 2], const uint32_t (&a)[TM], const uint32_t (&b)[TN / 2],
                                          const HalfConst& c) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const h2 w = as_h2(a[i]);
        const h2 ab = HI ? __builtin_shufflevector(w, w, 1, 1) : __builtin_shufflevector(w, w, 0, 0);
#pragma unroll
        for (int j = 0; j < TN / 2; ++j)
            acc[i][j] = PM == PM_IDENT ? __builtin_elementwise_fma(ab, as_h2(b[j]), acc[i][j]) : __builtin_elementwise_fma(q[i][j], c.kc, acc[i][j]);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// ... and their rounding to M + 1 bits
template <bool CLAMP, int TM, int TN, bool PRIO = (TM * TN > 4), bool MASK = true>
__device__ __forceinline__ void half_round(h2 (&acc)[TM][TN / 2], const HalfConst& c) {
    if (MASK) {
        issue_last<PRIO>();
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) acc[i][j] = as_h2(as_u32(acc[i][j]) & c.mask);
        __builtin_amdgcn_sched_barrier(0);
        issue_first<PRIO>();
    }
    if (CLAMP) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) {
                asm("v_pk_min_f16 %0, %0, %1" : "+v"(acc[i][j]) : "v"(c.rof));
                asm("v_pk_max_f16 %0, %0, %1" : "+v"(acc[i][j]) : "v"(c.nrof));
            }
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Second level of the chunked order: T <- Q_acc(T + S), S <- 0.
template <bool CLAMP, int TM, int TN>
__device__ __forceinline__ void half_level2(h2 (&top)[TM][TN / 2], h2 (&acc)[TM][TN / 2], const HalfConst& c) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) {
            top[i][j] = as_h2(as_u32(top[i][j] + acc[i][j]) & c.mask);
            acc[i][j] = as_h2(0u);
            if (CLAMP) {
                asm("v_pk_min_f16 %0, %0, %1" : "+v"(top[i][j]) : "v"(c.rof));
                asm("v_pk_max_f16 %0, %0, %1" : "+v"(top[i][j]) : "v"(c.nrof));
            }
        }
    __builtin_amdgcn_sched_barrier(0);
}

template <int TM, int BMP>
__device__ __forceinline__ void read_half_a(const uint32_t* As, int kp, int ty, uint32_t (&a)[TM]) {
    static_assert(TM >= 1 && TM <= 4, "rows per lane");
    if (TM >= 3) {
        const uint4 v = *reinterpret_cast<const uint4*>(As + kp * BMP + ty * 4);
        a[0] = v.x; a[TM > 1 ? 1 : 0] = v.y; a[TM > 2 ? 2 : 0] = v.z;
        if (TM == 4) a[TM - 1] = v.w;
    } else if (TM == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(As + kp * BMP + ty * 2);
        a[0] = v.x; a[TM - 1] = v.y;
    } else {
        a[0] = As[kp * BMP + ty];
    }
}

template <int TN, int BNP>
__device__ __forceinline__ void read_half_b(const uint32_t* Bs, int k, int tx, uint32_t (&b)[TN / 2]) {
    static_assert(TN == 2 || TN == 4, "columns per lane");
    if (TN == 4) {
        const uint2 v = *reinterpret_cast<const uint2*>(Bs + k * BNP + tx * 2);
        b[0] = v.x; b[TN / 2 - 1] = v.y;
    } else {
        b[0] = Bs[k * BNP + tx];
    }
}

// Decodes and stores the pieces of one k-tile.  dyn: also leaves the largest squared norm of a piece of A (low half) and of
// B, to 8 bits, rounded up, per wave.
template <int BM, int BN>
__device__ __forceinline__ void half_stage(const KParams& p, uint32_t* __restrict__ Ad, uint32_t* __restrict__ Bd, const uint4& ra, const uint4& rb,
                                           int tid, int tidb, bool dyn, uint32_t* __restrict__ norm) {
    uint32_t wa[8], wb[8];
    decode_half(ra, p.h_shift_a, p.h_keep_a, p.h_scale_a, wa);
    store_half_a<BM>(Ad, tid, wa);
    decode_half(rb, p.h_shift_b, p.h_keep_b, p.h_scale_b, wb);
    store_half_b<BN>(Bd, tidb, wb);
    if (dyn) {
        const uint32_t na = __float_as_uint(piece_norm2(wa)), nb = __float_as_uint(piece_norm2(wb));
        uint32_t m = ((na + 0xFFFFu) >> 16) | ((nb + 0xFFFFu) & 0xFFFF0000u);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = pk_max_u16(m, (uint32_t)__shfl_xor((int)m, o, 64));
        if ((tid & 63) == 0) norm[tid >> 6] = m;
    }
}

// 16-bit mask of a piece's non-zero codes, code 0 in bit 0
__device__ __forceinline__ uint32_t nonzero_codes(const uint4& v) {
    const uint32_t q[4] = {v.x, v.y, v.z, v.w};
    uint32_t b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = (((q[i] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) >> 7) & 0x01010101u;   // 1 per non-zero byte
    const uint32_t lo = __builtin_amdgcn_udot4(b[1], 0x80402010u, __builtin_amdgcn_udot4(b[0], 0x08040201u, 0u, false), false);
    const uint32_t hi = __builtin_amdgcn_udot4(b[3], 0x80402010u, __builtin_amdgcn_udot4(b[2], 0x08040201u, 0u, false), false);
    return lo | (hi << 8);
}

// The bound that follows the data costs a reduction per staged tile: only where the fixed one leaves less than half of the
// range (R_OF below 64 of the largest products).
__device__ __forceinline__ bool half_follows_data(const KParams& p) { return p.dyn_bound != 0 && 2.0f * p.fast_thresh < p.rof_a; }

// For how many of the next tiles of 32 steps (0 to 8) no sum of the wave can reach R_OF, or the end of FP16's range; mf: this lane's largest |S|.
struct HalfBound {
    float rof, thresh, grow, kcf;
    // grow: 32 of the largest products there are (thresh is rounded down; the factor covers the roundings here)
    __device__ __forceinline__ explicit HalfBound(const KParams& p)
        : rof(p.h_top), thresh(p.h_thresh), grow(1.0001f * (rof - thresh)), kcf((float)as_h2(p.h_kc).x) {}
    // whether n steps from here cannot
    __device__ __forceinline__ bool covers(float mf, int n) const { return __all(mf < rof - grow * ((float)n * 0x1p-5f)); }
    // ... nor parts of the current tile, by half_stage's norms of its pieces.  Cauchy-Schwarz: 16 products of a row's piece and a column's
    // piece add at most the product of their norms; a part's 32 steps are two pieces.  (The factor covers the roundings of the
    // norms and of this line.)
    __device__ __forceinline__ bool follows(float mf, const uint32_t* norms, int parts) const {
        const uint32_t m = pk_max_u16(pk_max_u16(norms[0], norms[1]), pk_max_u16(norms[2], norms[3]));
        const float n2 = __uint_as_float(m << 16) * __uint_as_float(m & 0xFFFF0000u);
        return __all(mf < rof - (float)parts * 2.0f * 1.001f * __builtin_sqrtf(n2) * kcf);
    }
    // norms: or null
    __device__ __forceinline__ int safe(float mf, const uint32_t* norms) const {
        if (__all(mf < thresh - 3.0f * grow)) return __all(mf < thresh - 7.0f * grow) ? 8 : 4;
        if (__all(mf < thresh)) return __all(mf < thresh - grow) ? 2 : 1;
        return norms && follows(mf, norms, 1) ? 1 : 0;
    }
};

// k-tiles whose pieces are in flight at a time: one for the large lane blocks (two measured the same); four for the small ones,
// whose tile takes less time than a load (64 x 1000 x 2048: 47 -> 45 us).
__host__ __device__ constexpr int half_depth(int TM, int TN) { return TM * TN <= 4 ? kTilesAhead : 1; }

}  // namespace lba
#endif

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
// every shape measured 3-8 % slower, with 5 to 8 waves per SIMD instead of 4 none faster, and an 8 x 4 lane block slower
// on every layer of ResNet-50.  Measured against the FP32 tile on the same grids: 8192 x 4096 x 1152 1819 -> 1573 us
// (6.4 cycles per chain and step), the ResNet-50 sweep 14.05 -> 11.92 ms, its 7 x 7 x 3 first convolution at batch 37 337 ->
// 250 us, the 64 x 1000 x 2048 classifier 61 -> 44 us, 3136 x 512 x 4608 of M4E3 codes 593 -> 520 us.

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

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ uint32_t as_u32(h2 h) { return __builtin_bit_cast(uint32_t, h); }
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
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
template <int PM, bool HI, int TM, int TN>
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
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) q[i][j] = as_h2(as_u32(q[i][j]) & c.maskp);
        __builtin_amdgcn_sched_barrier(0);
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
template <bool CLAMP, int TM, int TN>
__device__ __forceinline__ void half_round(h2 (&acc)[TM][TN / 2], const HalfConst& c) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) acc[i][j] = as_h2(as_u32(acc[i][j]) & c.mask);
    if (CLAMP) {
        __builtin_amdgcn_sched_barrier(0);
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

// 32 steps (16 pairs) from LDS, fully unrolled; operands are read AHEAD pairs of steps before their use.  A lane block of one
// or two pairs of chains takes the next step's products between a step's sums and their rounding: nothing else separates the
// dependent instructions there (the compiler puts a wait between a packed instruction and one that reads it at once).
template <int PM, int ORDER, bool CLAMP, int TM, int TN, int BMP, int BNP>
__device__ __forceinline__ void half_tile(h2 (&acc)[TM][TN / 2], h2 (&top)[TM][TN / 2], const uint32_t* As, const uint32_t* Bs,
                                          int tx, int ty, const HalfConst& c) {
    constexpr int AHEAD = TM * TN >= 12 ? 1 : (TM * TN >= 8 ? 2 : 4), SLOTS = AHEAD + 2;
    constexpr bool EARLY = TM * TN <= 4;
    uint32_t a[SLOTS][TM], b0[SLOTS][TN / 2], b1[SLOTS][TN / 2];
    h2 q[2][TM][TN / 2];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {
        read_half_a<TM, BMP>(As, s, ty, a[s]);
        read_half_b<TN, BNP>(Bs, 2 * s, tx, b0[s]);
        read_half_b<TN, BNP>(Bs, 2 * s + 1, tx, b1[s]);
    }
    if (EARLY) half_products<PM, false, TM, TN>(q[0], a[0], b0[0], c);
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int x = s % SLOTS;
        if (s + AHEAD < 16) {
            read_half_a<TM, BMP>(As, s + AHEAD, ty, a[(s + AHEAD) % SLOTS]);
            read_half_b<TN, BNP>(Bs, 2 * (s + AHEAD), tx, b0[(s + AHEAD) % SLOTS]);
            read_half_b<TN, BNP>(Bs, 2 * (s + AHEAD) + 1, tx, b1[(s + AHEAD) % SLOTS]);
        }
        if (!EARLY) half_products<PM, false, TM, TN>(q[0], a[x], b0[x], c);
        half_sums<PM, false, TM, TN>(acc, q[0], a[x], b0[x], c);
        if (EARLY) half_products<PM, true, TM, TN>(q[1], a[x], b1[x], c);
        half_round<CLAMP, TM, TN>(acc, c);
        if (!EARLY) half_products<PM, true, TM, TN>(q[1], a[x], b1[x], c);
        half_sums<PM, true, TM, TN>(acc, q[1], a[x], b1[x], c);
        if (EARLY && s < 15) half_products<PM, false, TM, TN>(q[0], a[(s + 1) % SLOTS], b0[(s + 1) % SLOTS], c);
        half_round<CLAMP, TM, TN>(acc, c);
        if (ORDER == LBA_ORDER_CHUNK16 && ((s + 1) & 7) == 0) half_level2<CLAMP, TM, TN>(top, acc, c);
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

// The bound that follows the data costs a reduction per staged tile: only where the fixed one leaves less than half of the
// range (R_OF below 64 of the largest products).
__device__ __forceinline__ bool half_follows_data(const KParams& p) { return p.dyn_bound != 0 && 2.0f * p.fast_thresh < p.rof_a; }

// For how many of the next tiles of 32 steps (0 to 4) no sum of the wave can reach R_OF; mf: this lane's largest |S|.
struct HalfBound {
    float rof, thresh, grow, kcf;
    // the planner's bound is in the FP32 tile's domain (R_UF at 2^-126); 2^112 moves it to R_UF at 2^-14.  grow: 32 of the
    // largest products there are (thresh is rounded down; the factor covers the roundings here)
    __device__ __forceinline__ explicit HalfBound(const KParams& p)
        : rof(p.rof_a * 0x1p112f), thresh(p.fast_thresh * 0x1p112f), grow(1.0001f * (rof - thresh)), kcf((float)as_h2(p.h_kc).x) {}
    // norms: half_stage's, for the current tile, or null
    __device__ __forceinline__ int safe(float mf, const uint32_t* norms) const {
        if (__all(mf < thresh)) return 1 + __all(mf < thresh - grow) + __all(mf < thresh - 2.0f * grow) + __all(mf < thresh - 3.0f * grow);
        if (!norms) return 0;
        // Cauchy-Schwarz: 16 products of a row's piece and a column's piece add at most the product of their norms; 32 steps
        // are two pieces.  (The factor covers the roundings of the norms and of this line.)
        const uint32_t m = pk_max_u16(pk_max_u16(norms[0], norms[1]), pk_max_u16(norms[2], norms[3]));
        const float n2 = __uint_as_float(m << 16) * __uint_as_float(m & 0xFFFF0000u);
        return __all(mf < rof - 2.0f * 1.001f * __builtin_sqrtf(n2) * kcf) ? 1 : 0;
    }
};

// k-tiles whose pieces are in flight at a time: one for the large lane blocks (two measured the same); four for the small ones,
// whose tile takes less time than a load (64 x 1000 x 2048: 47 -> 45 us).
__host__ __device__ constexpr int half_depth(int TM, int TN) { return TM * TN <= 4 ? kTilesAhead : 1; }

// The work of one workgroup: the BM x BN tile of C at (m0, n0).  smem: two stages.  Structure, clamp-free tiles and their
// bounds as in fast_body; AMODE as there, and 3, 4 below (every code format decodes alike).
template <int TM, int TN, int LX, int PM, int ORDER, int AMODE>
__device__ __forceinline__ void half_body(const KParams& p, uint32_t* __restrict__ smem, int m0, int n0) {
    using T = HalfTile<TM, TN, LX>;
    constexpr int BM = T::BM, BN = T::BN;
    static_assert(Stage<BM, HBK>::kPerLane == 1 && Stage<BN, HBK>::kPerLane == 1, "one piece per lane");
    static_assert(2 * T::STAGE <= 2 * 32 * 128, "two stages in 32 KB");
    const int tid = threadIdx.x;
    const int tx = tid % LX, ty = tid / LX;
    const int tidb = tid - Stage<BN, HBK>::kTailShift;
    const uint8_t* pA = p.A + (int64_t)blockIdx.z * p.stride_a;
    const uint8_t* pB = p.B + (int64_t)blockIdx.z * p.stride_b;
    float* pC = p.C + (int64_t)blockIdx.z * p.stride_c;

    set_flush_f32();
    set_round_zero_f16();
    set_flush_out_f16();

    HalfConst c;
    c.kc = as_h2(p.h_kc); c.rof = as_h2(p.h_rof); c.nrof = as_h2(p.h_rof ^ 0x80008000u); c.mask = p.h_mask_a; c.maskp = p.h_mask_p;
    asm volatile("" : "+v"(c.kc), "+v"(c.rof), "+v"(c.nrof), "+v"(c.mask), "+v"(c.maskp));

    h2 acc[TM][TN / 2], top[TM][TN / 2];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) { acc[i][j] = as_h2(0u); top[i][j] = as_h2(0u); }

    const int ntiles = (p.K + HBK - 1) / HBK;
    __shared__ uint32_t half_norm[2][4];                       // per stage and wave: largest squared norm of a piece of A (low half), of B
    const bool dyn = half_follows_data(p);
    // How the pieces come.  Aligned rows and im2col rows of whole 16-channel taps (AMODE 0, 2): one aligned load, zeroed at once
    // outside the operand.  Any other rows (AMODE 3, 4) and the small lane blocks: lba_piece.h, uncorrected loads that stay in
    // flight (C = 3 under a 7 x 7 filter: two loads a piece instead of sixteen, 279 -> 250 us).  Either kind of
    // code in the other's kernel, behind a uniform branch, cost the aligned shapes 1 to 4 %.
    constexpr bool SMALL = TM * TN <= 4, PIECES = SMALL || AMODE >= 3;
    static_assert(AMODE == 0 || AMODE == 2 || AMODE == 3 || AMODE == 4, "other operand formats decode alike: no AMODE of their own");
    constexpr bool conv = AMODE == 2 || AMODE == 4;
    const RowPieces<BM> sa(pA, conv ? 1 : p.M, p.K, conv ? 0 : m0, tid);
    const RowPieces<BN> sb(pB, p.N, p.K, n0, tidb);
    ConvPieces sc = {};
    ConvLane cl = {};
    if (PIECES && conv) sc = ConvPieces::make<BM>(pA, p, m0, tid);
    if (!PIECES && AMODE == 2) cl = conv_lane<BM, HBK>(pA, p, m0, tid);
    // pieces in flight: DEPTH tiles of them (1: asked for at the start of the tile before)
    constexpr int DEPTH = half_depth(TM, TN);
    uint4 ra[DEPTH], rc[DEPTH], rb[DEPTH];
    auto fetch = [&](int t, int d) {
        const int k0 = tile_start(t);
        if (PIECES) {
            if (conv) load_piece(sc, p, k0, ra[d], rc[d]);
            else      ra[d] = load_piece(sa, k0);
            rb[d] = load_piece(sb, k0);
        } else {
            ra[d] = AMODE == 2 ? fetch_taps(cl, p, k0) : fetch_aligned<BM>(pA, p.M, p.K, m0, k0, tid);
            rb[d] = fetch_aligned<BN>(pB, p.N, p.K, n0, k0, tidb);
        }
    };
    auto stage = [&](int t, int d) {
        const uint4 va = !PIECES ? ra[d] : (conv ? sc.codes(p, ra[d], rc[d], t * HBK) : sa.codes(ra[d], t * HBK));
        const uint4 vb = PIECES ? sb.codes(rb[d], t * HBK) : rb[d];
        const int st = t & 1;
        half_stage<BM, BN>(p, smem + st * T::STAGE, smem + st * T::STAGE + T::A_WORDS, va, vb, tid, tidb, dyn, half_norm[st]);
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) fetch(d, d);               // (a tile beyond K reads codes inside the operands that nothing uses)
    stage(0, 0);
    if (DEPTH > 1) fetch(DEPTH, 0);
    __syncthreads();

    const HalfBound bound(p);
    int safe_tiles = 0;
    for (int t0 = 0; t0 < ntiles; t0 += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int t = t0 + d;
            if (t >= ntiles) break;
            const uint32_t* As0 = smem + (t & 1) * T::STAGE;
            const uint32_t* Bs0 = As0 + T::A_WORDS;
            const bool more = (t + 1) < ntiles;
            if (DEPTH == 1 && (PIECES || more)) fetch(t + 1, 0);
            const int parts = p.K - t * HBK > 32 ? 2 : 1;      // steps beyond K are products of zeros: skipped 32 at a time
            for (int part = 0; part < parts; ++part) {
                const uint32_t* As = As0 + part * 16 * T::BMP;
                const uint32_t* Bs = Bs0 + part * 32 * T::BNP;
                if (safe_tiles == 0) {
                    uint32_t mx = 0u;
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN / 2; ++j)
                            mx = pk_max_u16(mx, as_u32(ORDER == LBA_ORDER_CHUNK16 ? top[i][j] : acc[i][j]) & 0x7FFF7FFFu);
                    safe_tiles = bound.safe(max_half(mx), dyn ? half_norm[t & 1] : nullptr);
                }
                if (safe_tiles > 0) {
                    --safe_tiles;
                    half_tile<PM, ORDER, false, TM, TN, T::BMP, T::BNP>(acc, top, As, Bs, tx, ty, c);
                } else {
                    half_tile<PM, ORDER, true, TM, TN, T::BMP, T::BNP>(acc, top, As, Bs, tx, ty, c);
                }
            }
            if (more) {
                constexpr int next = (DEPTH > 1) ? 1 : 0;
                stage(t + 1, (d + next) % DEPTH);
                if (DEPTH > 1) fetch(t + 1 + DEPTH, (d + next) % DEPTH);
            }
            __syncthreads();
        }
    }

    // C = S * 2^out_exp, zero written as +0
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + ty * TM + i;
        if (m >= p.M) continue;
        const int n = n0 + tx * TN;
        float v[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const h2 w = ORDER == LBA_ORDER_CHUNK16 ? top[i][j / 2] : acc[i][j / 2];
            const float s = (float)(j & 1 ? w.y : w.x);
            v[j] = __builtin_ldexpf(s, p.out_exp - 112) + 0.0f;    // -0 + 0 is +0
        }
        float* dst = pC + (int64_t)m * p.N + n;
        if (TN == 4 && p.c_vec && n + 3 < p.N) {
            *reinterpret_cast<f32x4_any*>(dst) = f32x4_any{v[0], v[1], v[TN - 2], v[TN - 1]};
        } else if (TN == 2 && p.c_vec && n + 1 < p.N) {
            *reinterpret_cast<f32x2_any*>(dst) = f32x2_any{v[0], v[1]};
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (n + j < p.N) dst[j] = v[j];
        }
    }
}

// The grids of lba_fast_kernel and lba_fast_mixed_kernel (the same tiles, numbered the same) on packed carriers.
// AMODE 0: row-major, 16-byte rows; 3: row-major, any K and alignment; 2: im2col rows, C % 16 == 0 and 16-byte rows; 4: any other.
template <int TM, int TN, int PM, int ORDER, int AMODE>
__global__ void __launch_bounds__(256, LBA_FAST_MIN_WAVES) lba_half_kernel(const KParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[2 * HalfTile<TM, TN, 16>::STAGE];
    half_body<TM, TN, 16, PM, ORDER, AMODE>(p, smem, blockIdx.x * 16 * TM, blockIdx.y * 16 * TN);
}

template <int PM, int ORDER, int AMODE>
__global__ void __launch_bounds__(256, LBA_FAST_MIN_WAVES) lba_half_mixed_kernel(const KParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[2 * HalfTile<4, 4, 16>::STAGE];
    const int b = blockIdx.x;
    if (b < p.mix_main) {                                      // uniform
        const int by = b / p.mix_gx_main, bx = b - by * p.mix_gx_main;
        half_body<4, 4, 16, PM, ORDER, AMODE>(p, smem, bx * 64, by * 64);
    } else if (b < p.mix_main + p.mix_half) {
        const int t = b - p.mix_main;
        const int by = t / p.mix_gx_half, bx = t - by * p.mix_gx_half;
        half_body<3, 4, 16, PM, ORDER, AMODE>(p, smem, p.mix_m_main + bx * 48, by * 64);
    } else {
        const int t = b - p.mix_main - p.mix_half;
        const int by = t / p.mix_gx_tail, bx = t - by * p.mix_gx_tail;
        if (p.mix_tail16) half_body<1, 2, 8, PM, ORDER, AMODE>(p, smem, p.mix_m_half + bx * 32, by * 16);   // uniform
        else              half_body<2, 2, 16, PM, ORDER, AMODE>(p, smem, p.mix_m_half + bx * 32, by * 32);
    }
}

}  // namespace lba
#endif

// lba_half_bwd.h -- the recompute call (forward chain + event planes) on the packed FP16 carriers of lba_half.h: floor
// rounding, Q_prod can flush, both orders.  Two chains per register; the event bits are collected two chains per register
// too, without the lane masks and carry-in adds of the FP32 kernel.
//
//   OF_k  <=>  |t| >= R_OF: the truncated sum's magnitude bits plus (0x8000 - bits of R_OF) carry into bit 15.
//   UF_k  <=>  the product was flushed with both operands non-zero, or 0 < |t| < R_UF.  The multiply runs with results flushed
//         (q = 0: flushed, or an operand is zero), the multiply-add with denormal results kept and denormal inputs read as
//         zero: t is a denormal number exactly when it underflows, and the next step reads it as the zero the quantizer
//         asks for.  A non-zero sum never rounds to zero there: with S != 0 it is a multiple of 2^-24 (S of M + 1 <= 11 bits
//         at 2^-14 or above, a product of at most 10 bits cancelling it), with S = 0 it is the product, at least 2^-14 * kc
//         (the planner admits kc >= 2^-10).  2|q| and 2|t| - 2 (a zero sum wraps to the top) are below 0x7FE exactly for
//         the two events, so one minimum and one add put "no event" into bit 15.  Steps with a zero operand are cleared
//         afterwards, a word at a time, from per-row masks of non-zero codes left by the staging.
//   Bit 15 of both halves of two registers enters a shift register of four bytes from the top: after 8 steps bit j of each byte is step j.
// A k-tile in which no sum can reach R_OF (HalfBound) has no overflow test.  Without an underflow plane such a tile is the forward call's
// (rows_body, lba_rows.h), and half_bwd_tile runs the others.
//
// What bounds it: VALU issue, eight and a half instructions for two chains with the underflow plane and a quiet tile (6.5 of them at
// half rate; full-rate ones of three waves hardly ever meet, so that their number counts: 1209 -> 1399 us with ands and adds for the
// underflow test, 11 instructions).  The FP32 kernel (compares to 64-bit masks, scalar logic, one carry-in add per chain and plane)
// takes 27 cycles per chain and step.  Measured against it, both planes of 4096 x 768 x 3072: 1703 -> 1396 us (2.4 GB of planes leave at
// 1.7 TB/s), with turns (lba_device.h) 1229, with the 32 steps unrolled 1210 (by four 1240), the flags of two registers gathered into
// one on their way to the shift register (8.5 instructions for 9; 11.5 for 13 where sums can reach R_OF) 1183 and, every sum loud,
// 1944 -> 1896.  Reading operands a step ahead, or two waves per SIMD instead of three, changed nothing.
#ifndef LBA_HALF_BWD_H_
#define LBA_HALF_BWD_H_

#include "lba_half.h"

namespace lba {

// FP16: denormal inputs read as zero, denormal results kept / both flushed (no memory clobber: everything that depends on
// the mode between two writes is volatile assembly itself)
__device__ __forceinline__ void half_keep_out()  { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 6, 2), 2\n\ts_nop 1"); }
__device__ __forceinline__ void half_flush_out() { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 6, 2), 1\n\ts_nop 1"); }
__device__ __forceinline__ void half_flush_all() { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 6, 2), 0\n\ts_nop 1" ::: "memory"); }

__device__ __forceinline__ uint32_t pk_add_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_add_u16_sat(uint32_t a, uint32_t b) {   // saturates at 0xFFFF
    uint32_t r;
    asm("v_pk_add_u16 %0, %1, %2 clamp" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
// shift register of four chains, a byte each, shifted by one already: bit 15 of the halves of y0 and y1 enters at the top
__device__ __forceinline__ uint32_t pk_shift_in(uint32_t w, uint32_t y0, uint32_t y1, uint32_t tops) {
    uint32_t r;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0xd8" : "=v"(r) : "v"(w), "v"(__builtin_amdgcn_perm(y1, y0, 0x07050301u)), "v"(tops));   // tops ? y : w
    return r;
}
// w[q]: steps 8 q to 8 q + 7 of four chains, a byte each -> w[c]: the 32 steps of chain c
__device__ __forceinline__ void bytes_to_chains(uint32_t& w0, uint32_t& w1, uint32_t& w2, uint32_t& w3) {
    const uint32_t a = __builtin_amdgcn_perm(w1, w0, 0x05010400u), b = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(w3, w2, 0x05010400u), d = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
    w0 = __builtin_amdgcn_perm(c, a, 0x05040100u); w1 = __builtin_amdgcn_perm(c, a, 0x07060302u);
    w2 = __builtin_amdgcn_perm(d, b, 0x05040100u); w3 = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

struct HalfBwdConst {
    h2 kc, rof, nrof;
    uint32_t mask, maskp;
    uint32_t absmask;          // the accumulator's mask without the sign
    uint32_t of_bias;          // 0x8000 - bits of R_OF
    uint32_t two, minus2, uf_bias;   // 2, -2, 0x8000 - 0x7FE
    uint32_t tops;             // 0x80808080
    __device__ __forceinline__ explicit HalfBwdConst(const KParams& p)
        : kc(as_h2(p.h_kc)), rof(as_h2(p.h_rof)), nrof(as_h2(p.h_rof ^ 0x80008000u)), mask(p.h_mask_a), maskp(p.h_mask_p), absmask(p.h_mask_a & 0x7FFF7FFFu),
          of_bias(pk_add_u16(0x80008000u, pk_add_u16(~p.h_rof, 0x00010001u))), two(0x00020002u), minus2(0xFFFEFFFEu), uf_bias(0x78027802u), tops(0x80808080u) {
        asm volatile("" : "+v"(kc), "+v"(rof), "+v"(nrof), "+v"(mask), "+v"(maskp), "+v"(absmask), "+v"(of_bias), "+v"(two), "+v"(minus2), "+v"(uf_bias), "+v"(tops));
    }
};

// 32 steps with event bits: word [i][j] of chain (i, j) gets step k in bit k (of: 1 = overflow; uf: 1 = underflow or a zero
// operand, cleared by the caller).  of2 / uf2: the two chunks' bits enter the second-level words at bits pos, pos + 1.
// read_a(k / 2, words of the rows), read_b(k, words of the columns).
template <int PM, int ORDER, bool UF, bool QUIET, int TM, int TN, bool PRIO, class ReadA, class ReadB>
__device__ __forceinline__ void half_bwd_tile(h2 (&acc)[TM][TN / 2], h2 (&top)[TM][TN / 2], uint32_t (&of)[TM][TN], uint32_t (&uf)[TM][TN],
                                              uint32_t (&of2)[TM][TN], uint32_t (&uf2)[TM][TN], int pos, ReadA read_a, ReadB read_b,
                                              const HalfBwdConst& c) {
    constexpr int NJ = TN / 2, G = TM * NJ / 2;                // G: groups of two registers, four chains
    static_assert(TM * NJ % 2 == 0, "registers in twos");
    uint32_t wo[G], wu[G];
#pragma unroll
    for (int g = 0; g < G; ++g) { wo[g] = 0u; wu[g] = 0u; }
    issue_first<PRIO>();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            uint32_t a[TM], b[2][NJ];
            read_a(8 * h + s, a);
            read_b(16 * h + 2 * s, b[0]);
            read_b(16 * h + 2 * s + 1, b[1]);
            uint32_t q[2][TM][NJ];
            // both steps' products under one mode: below Q_prod's R_UF they are flushed
            if (UF) half_flush_out();
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    asm volatile("v_pk_mul_f16 %0, %1, %2 op_sel_hi:[0,1]" : "=v"(q[0][i][j]) : "v"(a[i]), "v"(b[0][j]));
                    asm volatile("v_pk_mul_f16 %0, %1, %2 op_sel:[1,0]" : "=v"(q[1][i][j]) : "v"(a[i]), "v"(b[1][j]));
                }
            if (UF) half_keep_out();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (PM == PM_TRUNC) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j) q[u][i][j] &= c.maskp;
                }
                uint32_t t[TM][NJ];
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) asm volatile("v_pk_fma_f16 %0, %1, %2, %3" : "=v"(t[i][j]) : "v"(q[u][i][j]), "v"(c.kc), "v"(acc[i][j]));
                // phase by phase over the lane's chains, as the forward tile
#define LBA_GROUP for (int g = 0; g < G; ++g)
#define LBA_EACH for (int i = 0; i < TM; ++i) _Pragma("unroll") for (int j = 0; j < NJ; ++j)
                __builtin_amdgcn_sched_barrier(0);
                issue_last<PRIO>();
                _Pragma("unroll") LBA_EACH acc[i][j] = as_h2(t[i][j] & c.mask);
                if (!QUIET) { _Pragma("unroll") LBA_GROUP wo[g] >>= 1; }   // full-rate as well
                if (UF) { _Pragma("unroll") LBA_GROUP wu[g] >>= 1; }
                __builtin_amdgcn_sched_barrier(0);
                issue_first<PRIO>();
                if (!QUIET) {
                    _Pragma("unroll") LBA_EACH asm("v_pk_min_f16 %0, %0, %1" : "+v"(acc[i][j]) : "v"(c.rof));
                    _Pragma("unroll") LBA_EACH asm("v_pk_max_f16 %0, %0, %1" : "+v"(acc[i][j]) : "v"(c.nrof));
                    __builtin_amdgcn_sched_barrier(0);
                    uint32_t y[TM][NJ];
                    _Pragma("unroll") LBA_EACH y[i][j] = (t[i][j] & c.absmask) + c.of_bias;   // at most 0x7FFF + 0x8000: no carry between the halves
                    __builtin_amdgcn_sched_barrier(0);
                    _Pragma("unroll") LBA_GROUP wo[g] = pk_shift_in(wo[g], y[2 * g / NJ][2 * g % NJ], y[(2 * g + 1) / NJ][(2 * g + 1) % NJ], c.tops);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (UF) {
                    _Pragma("unroll") LBA_EACH asm("v_pk_mad_u16 %0, %0, %1, %2" : "+v"(t[i][j]) : "v"(c.two), "v"(c.minus2));
                    _Pragma("unroll") LBA_EACH q[u][i][j] = pk_add_u16(q[u][i][j], q[u][i][j]);
                    __builtin_amdgcn_sched_barrier(0);
                    _Pragma("unroll") LBA_EACH t[i][j] = pk_min_u16(q[u][i][j], t[i][j]);
                    __builtin_amdgcn_sched_barrier(0);
                    _Pragma("unroll") LBA_EACH t[i][j] = pk_add_u16_sat(t[i][j], c.uf_bias);
                    __builtin_amdgcn_sched_barrier(0);
                    _Pragma("unroll") LBA_GROUP wu[g] = pk_shift_in(wu[g], t[2 * g / NJ][2 * g % NJ], t[(2 * g + 1) / NJ][(2 * g + 1) % NJ], c.tops);
                    __builtin_amdgcn_sched_barrier(0);
                }
#undef LBA_EACH
#undef LBA_GROUP
            }
            if (s % 4 == 3) {                                  // eight steps
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int ch = 4 * g + 2 * h + s / 4;
                    of[ch / TN][ch % TN] = wo[g];
                    if (UF) uf[ch / TN][ch % TN] = wu[g];
                }
            }
        }
        if (ORDER == LBA_ORDER_CHUNK16) {                      // the mode is the multiply-add's (UF) or the forward call's
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    uint32_t t;
                    asm volatile("v_pk_add_f16 %0, %1, %2" : "=v"(t) : "v"(top[i][j]), "v"(acc[i][j]));
                    top[i][j] = as_h2(t & c.mask);
                    acc[i][j] = as_h2(0u);
                    if (!QUIET) {
                        asm("v_pk_min_f16 %0, %0, %1" : "+v"(top[i][j]) : "v"(c.rof));
                        asm("v_pk_max_f16 %0, %0, %1" : "+v"(top[i][j]) : "v"(c.nrof));
                        const uint32_t y = pk_add_u16(t & c.absmask, c.of_bias);
                        of2[i][2 * j] |= ((y >> 15) & 1u) << (pos + h);
                        of2[i][2 * j + 1] |= (y >> 31) << (pos + h);
                    }
                    if (UF) {                                  // 0 < |t| < R_UF
                        uint32_t t2;
                        asm("v_pk_mad_u16 %0, %1, %2, %3" : "=v"(t2) : "v"(t), "v"(c.two), "v"(c.minus2));
                        const uint32_t y = ~pk_add_u16_sat(t2, c.uf_bias);
                        uf2[i][2 * j] |= ((y >> 15) & 1u) << (pos + h);
                        uf2[i][2 * j + 1] |= (y >> 31) << (pos + h);
                    }
                }
        }
    }
#pragma unroll
    for (int ch = 0; ch < TM * TN; ch += 4) {
        const auto each = [&](uint32_t (&w)[TM][TN]) {
            bytes_to_chains(w[ch / TN][ch % TN], w[(ch + 1) / TN][(ch + 1) % TN], w[(ch + 2) / TN][(ch + 2) % TN], w[(ch + 3) / TN][(ch + 3) % TN]);
        };
        each(of);
        if (UF) {
            each(uf);
#pragma unroll
            for (int u = ch; u < ch + 4; ++u) uf[u / TN][u % TN] = ~uf[u / TN][u % TN];   // bits say "no event": inverted
        }
    }
    issue_last<PRIO>();
}

// Stores a lane's words (one per chain, first step in bit 0) as word `word` of a plane; non-temporal, see store_event_words.
// 16 lanes a row.  ENDS (N no multiple of 4): where the matrix ends inside a lane's columns, that lane stores the last TN words of the
// row, some of them its neighbour's (which stores the same), so that a row still leaves by one store an instruction: word by word the end
// of a row went to memory as partial lines of its own.  Both planes, us, before -> so: 45658 x 106 x 729 710 -> 596 (104 columns 565),
// 30000 x 99 x 640 420 -> 364, 20000 x 250 x 500 413 -> 381.  Kernels of their own (AMODE 3): the address and masks beside the ordinary
// stores cost these 1 % (45658 x 128 x 729 560 -> 565).  Not the whole of it: a tile that holds no more than one lane's columns (width 64 n + 1 to
// 64 n + 3, 32 n + 1 in small tiles) has no neighbour to take words from and stores them one by one, and so do im2col rows (AMODE 2)
// and the overflow plane alone (lba_rows.h).  With truncated products, chains of 33 to 64 steps and one round and a third of workgroups,
// it loses where C is stored too (2328 x 2243 x 46 63 -> 69; without C 60 -> 59, 1164 rows 42 -> 41, 160 steps 139 -> 135).
template <int TM, int TN, bool ENDS>
__device__ __forceinline__ void store_half_words(uint32_t* __restrict__ plane, int word, const uint32_t (&w)[TM][TN], int m0, int n0,
                                                 int tx, int ty, const KParams& p) {
    static_assert(TN == 4 || TN == 2, "4 or 2 outputs per lane along n");
    const int left = p.N - n0, over = p.N & (TN - 1);          // columns from n0; columns of the lane in which the matrix ends
    const int n = n0 + tx * TN;
    uint32_t* row = plane + ((int64_t)word * p.M + m0 + ty * TM) * p.N + n;
    if (ENDS && p.c_vec && over != 0 && left > TN && left < 16 * TN) {   // uniform
        const bool last = n < p.N && n + TN - 1 >= p.N;
        row -= last ? TN - over : 0;
        const uint32_t by1 = last && over == 1 ? ~0u : 0u, by2 = last && over == 2 ? ~0u : 0u, by3 = last && over == 3 ? ~0u : 0u;
#pragma unroll
        for (int i = 0; i < TM; ++i, row += p.N) {
            uint32_t x[2 * TN];                                // the neighbour's words and the lane's
#pragma unroll
            for (int j = 0; j < TN; ++j) { x[j] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[i][j], 0x111, 0xF, 0xF, true); x[TN + j] = w[i][j]; }
            uint32_t v[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {                     // word j + over of the eight (masks: a choice between them went to scratch memory)
                const uint32_t one = x[j + 1], two = x[TN == 4 ? j + 2 : j], three = x[TN == 4 ? j + 3 : j], own = x[TN + j];
                v[j] = (one & by1) | (~by1 & ((two & by2) | (~by2 & ((three & by3) | (~by3 & own)))));
            }
            if (m0 + ty * TM + i < p.M && n < p.N) {
                if (TN == 4) __builtin_nontemporal_store(u32x4_any{v[0], v[1], v[TN - 2], v[TN - 1]}, reinterpret_cast<u32x4_any*>(row));
                else         __builtin_nontemporal_store(u32x2_any{v[0], v[1]}, reinterpret_cast<u32x2_any*>(row));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + ty * TM + i;
        if (m >= p.M) continue;
        uint32_t* dst = plane + ((int64_t)word * p.M + m) * p.N + n;
        if (TN == 4 && p.c_vec && n + 3 < p.N) {
            __builtin_nontemporal_store(u32x4_any{w[i][0], w[i][1], w[i][TN - 2], w[i][TN - 1]}, reinterpret_cast<u32x4_any*>(dst));
        } else if (TN == 2 && p.c_vec && n + 1 < p.N) {
            __builtin_nontemporal_store(u32x2_any{w[i][0], w[i][1]}, reinterpret_cast<u32x2_any*>(dst));
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (n + j < p.N) __builtin_nontemporal_store(w[i][j], dst + j);
        }
    }
}

// mark_bricks (lba_device.h) for words whose first step is bit 0 and whose steps beyond K are cleared; word w.
template <int TM, int TN>
__device__ __forceinline__ void mark_bricks_lsb(const uint32_t (&of)[TM][TN], int m0, int n0, int w, int tx, int ty, const KParams& p) {
    uint32_t any = 0u;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            if (m0 + ty * TM + i < p.M && n0 + tx * TN + j < p.N) any |= of[i][j];
    mark_bricks_of_wave<TM, TN>(any, m0, n0, w, tx, ty, p);
}

// The recompute call with an underflow plane (without one: rows_body, lba_rows.h).  AMODE 0: rows of A, 2: im2col rows, 3: rows of A, N no
// multiple of 4.  TURNS: not where a wave has its SIMD to itself.
template <int TM, int TN, int PM, int ORDER, int AMODE, bool TURNS = (TM * TN > 4)>
__device__ __forceinline__ void half_bwd_body(const KParams& p, uint32_t* __restrict__ smem, int m0, int n0) {
    using T = HalfTile<TM, TN, 16>;
    constexpr int BM = T::BM, BN = T::BN, NJ = TN / 2;
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int tidb = tid - Stage<BN, HBK>::kTailShift;

    set_flush_f32();
    set_round_zero_f16();
    set_flush_out_f16();

    const HalfBwdConst c(p);
    h2 acc[TM][NJ], top[TM][NJ];
    uint32_t of2[TM][TN], uf2[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) { acc[i][j] = as_h2(0u); top[i][j] = as_h2(0u); }
#pragma unroll
        for (int j = 0; j < TN; ++j) { of2[i][j] = 0u; uf2[i][j] = 0u; }
    }

    const int ntiles = (p.K + HBK - 1) / HBK;
    __shared__ uint32_t half_norm[2][4];
    // non-zero codes: 64 bits per row of A and per column of B and stage, 16 per piece
    __shared__ __attribute__((aligned(8))) uint16_t nza[2][BM][4], nzb[2][BN][4];
    const bool dyn = half_follows_data(p);
    const RowPieces<BM> sa(p.A, AMODE == 2 ? 1 : p.M, p.K, AMODE == 2 ? 0 : m0, tid);
    const RowPieces<BN> sb(p.B, p.N, p.K, n0, tidb);
    ConvPieces sc = {};
    if (AMODE == 2) sc = ConvPieces::make<BM>(p.A, p, m0, tid);
    uint4 ra, rc, rb;
    auto fetch = [&](int t) {
        const int k0 = tile_start(t);
        if (AMODE == 2) load_piece(sc, p, k0, ra, rc);
        else            ra = load_piece(sa, k0);
        rb = load_piece(sb, k0);
    };
    auto stage = [&](int t) {
        const uint4 va = AMODE == 2 ? sc.codes(p, ra, rc, t * HBK) : sa.codes(ra, t * HBK);
        const uint4 vb = sb.codes(rb, t * HBK);
        const int st = t & 1;
        half_stage<BM, BN>(p, smem + st * T::STAGE, smem + st * T::STAGE + T::A_WORDS, va, vb, tid, tidb, dyn, half_norm[st]);
        {
            if (tid < Stage<BM, HBK>::kChunks) nza[st][tid % BM][tid / BM] = (uint16_t)nonzero_codes(va);
            if (tidb >= 0 && tidb < Stage<BN, HBK>::kChunks) nzb[st][tidb % BN][tidb / BN] = (uint16_t)nonzero_codes(vb);
        }
    };
    fetch(0);
    stage(0);
    __syncthreads();

    const HalfBound bound(p);
    const int words = (p.K + 31) >> 5;
    int safe_tiles = 0;
    for (int t = 0; t < ntiles; ++t) {
        const uint32_t* As0 = smem + (t & 1) * T::STAGE;
        const uint32_t* Bs0 = As0 + T::A_WORDS;
        const bool more = (t + 1) < ntiles;
        fetch(t + 1);
        const int parts = p.K - t * HBK > 32 ? 2 : 1;
        for (int part = 0; part < parts; ++part) {
            const uint32_t* As = As0 + part * 16 * T::BMP;
            const uint32_t* Bs = Bs0 + part * 32 * T::BNP;
            auto read_a = [&](int k, uint32_t (&a)[TM]) { read_half_a<TM, T::BMP>(As, k, ty, a); };
            auto read_b = [&](int k, uint32_t (&b)[NJ]) { read_half_b<TN, T::BNP>(Bs, k, tx, b); };
            const int w = 2 * t + part;                        // plane word of this part's steps
            if (safe_tiles == 0) {
                uint32_t mx = 0u;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        mx = pk_max_u16(mx, as_u32(ORDER == LBA_ORDER_CHUNK16 ? top[i][j] : acc[i][j]) & 0x7FFF7FFFu);
                safe_tiles = bound.safe(max_half(mx), dyn ? half_norm[t & 1] : nullptr);
            }
            uint32_t of[TM][TN], uf[TM][TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) { of[i][j] = 0u; uf[i][j] = 0u; }
            const int pos = 2 * (w & 15);
            const bool quiet = safe_tiles > 0;
            if (quiet) {
                --safe_tiles;
                half_bwd_tile<PM, ORDER, true, true, TM, TN, TURNS>(acc, top, of, uf, of2, uf2, pos, read_a, read_b, c);
            } else {
                half_bwd_tile<PM, ORDER, true, false, TM, TN, TURNS>(acc, top, of, uf, of2, uf2, pos, read_a, read_b, c);
                const int valid = p.K - 32 * w;                // a saturated sum stays at R_OF beyond K
                if (valid < 32) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) of[i][j] &= (1u << valid) - 1u;
                }
                if (ORDER == LBA_ORDER_SEQ && p.map_dx) mark_bricks_lsb<TM, TN>(of, m0, n0, w, tx, ty, p);
            }
            if (p.of_mask) store_half_words<TM, TN, AMODE == 3>(p.of_mask, w, of, m0, n0, tx, ty, p);
            if (p.uf_mask) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const uint32_t na = *reinterpret_cast<const uint32_t*>(&nza[t & 1][ty * TM + i][2 * part]);
#pragma unroll
                    for (int j = 0; j < TN; ++j) uf[i][j] &= na & *reinterpret_cast<const uint32_t*>(&nzb[t & 1][tx * TN + j][2 * part]);
                }
                store_half_words<TM, TN, AMODE == 3>(p.uf_mask, w, uf, m0, n0, tx, ty, p);
            }
            if (ORDER == LBA_ORDER_CHUNK16 && ((w & 15) == 15 || w == words - 1)) {
                // two chunks per word: a second-level word is complete after 16 of them
                const int left = ((p.K + 15) >> 4) - 32 * (w >> 4);
                const uint32_t vmask = left >= 32 ? 0xFFFFFFFFu : (1u << left) - 1u;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) { of2[i][j] &= vmask; uf2[i][j] &= vmask; }
                if (p.of_mask2) store_half_words<TM, TN, AMODE == 3>(p.of_mask2, w >> 4, of2, m0, n0, tx, ty, p);
                if (p.uf_mask2) store_half_words<TM, TN, AMODE == 3>(p.uf_mask2, w >> 4, uf2, m0, n0, tx, ty, p);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) { of2[i][j] = 0u; uf2[i][j] = 0u; }
            }
        }
        if (more) stage(t + 1);
        __syncthreads();
    }
    if (!p.C) return;
    half_flush_all();                                          // a denormal sum reads as zero
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + ty * TM + i, n = n0 + tx * TN;
        if (m >= p.M) continue;
        float v[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const uint32_t w = as_u32(ORDER == LBA_ORDER_CHUNK16 ? top[i][j / 2] : acc[i][j / 2]);
            float s;
            asm volatile("v_cvt_f32_f16 %0, %1" : "=v"(s) : "v"(j & 1 ? w >> 16 : w));
            v[j] = __builtin_ldexpf(s, p.out_exp - 112) + 0.0f;
        }
        float* dst = p.C + (int64_t)m * p.N + n;
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

}  // namespace lba
#endif

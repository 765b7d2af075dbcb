// lba_rows.h -- the forward tile on packed FP16 carriers (lba_half.h has the arithmetic): groups of lanes that own rows of A.
//
// What bounds it: VALU issue, so the two things it does are fewer instructions and a better issue rate.
//
// Steps whose code of A is zero are not run.  A product of zero leaves the sum as it is (Q_acc(S + 0) = S: S is a value of Q_acc
// already), so such a step is the identity whatever the other operand, and half of what a layer with a ReLU before it does is
// such steps.  The chains of a register pair share a row of A, so the 8 lanes of a row can go through a list of its non-zero codes
// (value and place of the code's row of B in one word), each row of the wave its own; a wave runs as many steps as its longest
// list.  The wave builds the lists itself (one compare, a count of the lanes below and one store per row of 64 codes), per
// k-tile and where they save enough: ReLU rows run 38 of 64 steps.  Codes without zeros cost a test of a quarter of them.
// Which steps run depends on the data, the result does not.
//
// Waves take turns by the rate of their instructions.  A full-rate instruction (the mask) issues in half the time of a packed
// one only when another wave has one too; with waves at random places of their steps it mostly has no partner and takes as long.
// Packed instructions run at priority 1 and the masks at priority 0, so waves gather at their masks (issue-rate probe: 12.1 ->
// 10.9 cycles per register and step).  A lone wave per SIMD (the smallest tiles, lba_half_alone.hip) has nobody to wait for and keeps one
// priority.
//
// Measured (us), 16 chains per lane in 4 x 4 blocks / rows without lists / with; no zeros, then half of A's codes zero:
//   8192 x 512 x 2304    447 -> 394,  447 -> 394 -> 329
//   50176 x 128 x 1152   319 -> 294,  319 -> 294 -> 242
//   12544 x 256 x 2304   335 -> 309,  335 -> 309 -> 258
//   200704 x 64 x 64      42 ->  41,   42 ->  41 ->  35
// and without the priorities 433 and 362 for the first shape.  ResNet-50 at batch 64: 11.96 -> 9.33 ms.
#ifndef LBA_ROWS_H_
#define LBA_ROWS_H_

#include "lba_half_bwd.h"
#include "lba_list_index.h"

namespace lba {

template <int T>
__device__ __forceinline__ void read_words(const uint32_t* s, uint32_t (&b)[T]) {
    static_assert(T == 1 || T == 2 || T == 4, "words per lane");
    if (T == 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(s);
        b[0] = v.x; b[T > 1 ? 1 : 0] = v.y; b[T > 2 ? 2 : 0] = v.z; b[T - 1] = v.w;
    } else if (T == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(s);
        b[0] = v.x; b[T - 1] = v.y;
    } else {
        b[0] = s[0];
    }
}

// A list's first 2 U entries.
template <int U>
struct ListHead {
    uint32_t e[U], f[U];
    static __device__ __forceinline__ void read(const uint32_t* list, uint32_t (&e)[U]) {
#pragma unroll
        for (int u = 0; u < U; u += 4) { uint32_t x[4]; read_words<4>(list + u, x); e[u] = x[0]; e[u + 1] = x[1]; e[u + 2] = x[2]; e[u + 3] = x[3]; }
    }
    __device__ __forceinline__ explicit ListHead(const uint32_t* list) { read(list, e); read(list + U, f); }
};

// U steps: entries e with their rows of B in b; the rows of the next entries f are asked for as the registers of a step become
// free, and the entries after those when the last of e is used.
template <int PM, bool CLAMP, bool MASK, int T, int U>
__device__ __forceinline__ void list_round(h2 (&acc)[1][T / 2], uint32_t (&e)[U], const uint32_t (&f)[U], uint32_t (&b)[U][T / 2],
                                           const uint32_t* after, const char* Bb, const HalfConst& c) {
    constexpr int W = T / 2;
    h2 q[1][W];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t a1[1] = {e[u]};
        half_products<PM, false, 1, T, true>(q, a1, b[u], c);
        half_sums<PM, false, 1, T>(acc, q, a1, b[u], c);
        if (u == U - 1) ListHead<U>::read(after, e);
        read_words<W>(reinterpret_cast<const uint32_t*>(Bb + (f[u] >> 16)), b[u]);
        half_round<CLAMP, 1, T, true, MASK>(acc, c);
    }
}

// The steps of a list of n entries, a multiple of U (it is read on for 2 U more).
template <int PM, bool CLAMP, bool MASK, int T, int U>
__device__ __forceinline__ void list_steps(h2 (&sums)[T / 2], ListHead<U>& h, const uint32_t* list, const char* Bb, int n, const HalfConst& c) {
    constexpr int W = T / 2;
    uint32_t b[U][W];
    h2 acc[1][W];
#pragma unroll
    for (int j = 0; j < W; ++j) acc[0][j] = sums[j];
#pragma unroll
    for (int u = 0; u < U; ++u) read_words<W>(reinterpret_cast<const uint32_t*>(Bb + (h.e[u] >> 16)), b[u]);
    const uint32_t* const after = list + 2 * U;
    issue_first<MASK>();
    walk_list<U>(n, [&](int i) { list_round<PM, CLAMP, MASK, T, U>(acc, h.e, h.f, b, after + i, Bb, c); },
                 [&](int i) { list_round<PM, CLAMP, MASK, T, U>(acc, h.f, h.e, b, after + i, Bb, c); });
    issue_last<MASK>();
#pragma unroll
    for (int j = 0; j < W; ++j) sums[j] = acc[0][j];
}

// 32 steps (16 pairs) of S sets of rows, fully unrolled, TN columns a lane.  arow: the lane's row of the first set (the next
// set's 8 rows on); Bs: the lane's words of the first step, BROW words a step.
template <int PM, int ORDER, bool CLAMP, bool MASK, bool LONE, int AHEAD, int S, int TN, int BROW, int PITCH>
__device__ __forceinline__ void rows_tile(h2 (&acc)[S][TN / 2], h2 (&top)[S][TN / 2], const uint32_t* arow, const uint32_t* Bs, const HalfConst& c) {
    constexpr int W = TN / 2;
    constexpr int SLOTS = AHEAD + 2;
    constexpr bool EARLY = LONE;
    uint32_t a[S][16], b0[SLOTS][W], b1[SLOTS][W];
    h2 q[2][S][W];
    auto read_a = [&](int s) {                                 // four pairs of steps
#pragma unroll
        for (int i = 0; i < S; ++i) {
            uint32_t x[4];
            read_words<4>(arow + i * 8 * PITCH + s, x);
#pragma unroll
            for (int j = 0; j < 4; ++j) a[i][s + j] = x[j];
        }
    };
    auto a_of = [&](int s, uint32_t (&x)[S]) {
#pragma unroll
        for (int i = 0; i < S; ++i) x[i] = a[i][s];
    };
    read_a(0);
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {
        read_words<W>(Bs + 2 * s * BROW, b0[s]);
        read_words<W>(Bs + (2 * s + 1) * BROW, b1[s]);
    }
    uint32_t x[S], y[S];
    a_of(0, x);
    issue_first<MASK && !EARLY>();
    if (EARLY) half_products<PM, false, S, TN, MASK && !LONE>(q[0], x, b0[0], c);
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int k = s % SLOTS;
        if (s % 4 == 2 && s < 12) read_a(s + 2);
        if (s + AHEAD < 16) {
            read_words<W>(Bs + 2 * (s + AHEAD) * BROW, b0[(s + AHEAD) % SLOTS]);
            read_words<W>(Bs + (2 * (s + AHEAD) + 1) * BROW, b1[(s + AHEAD) % SLOTS]);
        }
        a_of(s, x);
        if (!EARLY) half_products<PM, false, S, TN, MASK && !LONE>(q[0], x, b0[k], c);
        half_sums<PM, false, S, TN>(acc, q[0], x, b0[k], c);
        if (EARLY) half_products<PM, true, S, TN, MASK && !LONE>(q[1], x, b1[k], c);
        half_round<CLAMP, S, TN, MASK && !LONE, MASK>(acc, c);
        if (!EARLY) half_products<PM, true, S, TN, MASK && !LONE>(q[1], x, b1[k], c);
        half_sums<PM, true, S, TN>(acc, q[1], x, b1[k], c);
        if (EARLY && s < 15) { a_of(s + 1, y); half_products<PM, false, S, TN, MASK && !LONE>(q[0], y, b0[(s + 1) % SLOTS], c); }
        half_round<CLAMP, S, TN, MASK && !LONE, MASK>(acc, c);
        if (ORDER == LBA_ORDER_CHUNK16 && ((s + 1) & 7) == 0) half_level2<CLAMP, S, TN>(top, acc, c);
    }
    issue_last<MASK && !EARLY>();
}

typedef uint16_t __attribute__((may_alias)) u16_any;

// A lane's pieces of a row of a matrix whose rows are 16-byte aligned and at least 16 codes long (K % 16 == 0).  A row beyond the matrix reads its first row:
// what comes of it is not stored.
struct AlignedRow {
    const uint8_t* row;
    int last, kq, K;           // the last piece of the row; the lane's first
    __device__ __forceinline__ AlignedRow(const uint8_t* G, int rows, int K_, int r, int kq_) : row(G + (int64_t)(r >= 0 && r < rows ? r : 0) * K_), last(K_ - 16), kq(kq_), K(K_) {}
    // the piece of the tile at k0: zero beyond K
    __device__ __forceinline__ uint4 codes(const uint4& v, int k0) const {
        const bool in = k0 + kq < K;
        return make_uint4(in ? v.x : 0u, in ? v.y : 0u, in ? v.z : 0u, in ? v.w : 0u);
    }
};
__device__ __forceinline__ uint4 load_aligned(const AlignedRow& s, int k0) {
    return *reinterpret_cast<const uint4*>(s.row + min(k0 + s.kq, s.last));
}

// mark_bricks (lba_device.h) for the rows of a wave: RW rows inside one group of 32, 8 TN columns (two groups of 32 when TN = 8), first
// step in bit 0 and steps beyond K cleared; word w of the plane.
template <int RW, int TN>
__device__ __forceinline__ void mark_bricks_of_rows(const uint32_t (&of)[RW / 8][TN], int m0, int n0, int w, const KParams& p) {
    const int lane = threadIdx.x & 63, first = m0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * RW;
    uint32_t any = 0u;
#pragma unroll
    for (int i = 0; i < RW / 8; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            if (first + 8 * i + (lane >> 3) < p.M && n0 + (lane & 7) * TN + j < p.N) any |= of[i][j];
    const uint64_t dirty = __builtin_amdgcn_ballot_w64(any != 0u);
    if (dirty == 0) return;                                    // uniform; the usual case
    if (lane == 0) {
        const int64_t kb = w >> 3;
        uint8_t* bw = p.map_dw + (kb * p.map_rbw + (n0 >> 7)) * p.map_sbw + (first >> 5);
        if (!*bw) *bw = 1;                                     // racing stores write the same value
        uint8_t* bx = p.map_dx + (kb * p.map_rbx + (first >> 7)) * p.map_sbx + (n0 >> 5);
        const uint64_t low = TN == 8 ? 0x0F0F0F0F0F0F0F0Full : ~0ull;   // lanes whose columns lie in the first group
        if ((dirty & low) && !*bx) *bx = 1;
        if (TN == 8 && (dirty & ~low) && !bx[1]) bx[1] = 1;
    }
}

// Sums beyond FP16's range (accumulators of E >= 5), in FP32 at R_UF = 2^-126: the products of two chains stay packed, v_fma_mix_f32 adds
// one half of them to an FP32 sum (exactly, rounded once toward zero, flushed below R_UF), then the mask and, where R_OF is near, the
// clamp of the FP32 step.  No operand is converted, and the masks take turns with the rest as in the packed tile: 7.1 cycles per
// chain and step in the issue-rate probe at four waves per SIMD (FP32 step 6.8, packed step 5.6).
// All sums beyond the range, lba_fast_kernel / operands converted to FP32, four steps at a time and to the end of the chain / here, us:
//   4096 x 1024 x 2048   M7E6  463 / 1140 /  471, half of A's codes zero 463 /  840 / 386
//   4096 x 4096 x 4096   M7E6 3201 /10000 / 3343, ...                   3200 / 6489 /2613; M10E5, products of both signs 3238 / 3772 /2625
//   64 x 1000 x 2048     M7E6   61 /   86 /   62, ...                     61 /   71 /  56
// M10E5, where every sum saturates: 491 / 1252 / 528 for the first shape (the clamp has the same price for both, beside fewer instructions).
struct BeyondConst {
    float kc, rof, nrof;       // kc * 2^-112 (kc < 2^-14 never gets here: products below 4 carry no sum of 11 bits past 8192)
    uint32_t mask;
    __device__ __forceinline__ explicit BeyondConst(const KParams& p) : kc(p.kc * 0x1p-112f), rof(p.rof_a), nrof(-p.rof_a), mask(p.mask_a) {
        asm volatile("" : "+v"(kc), "+v"(rof), "+v"(nrof), "+v"(mask));
    }
};

// a step's products added to the sums, unrounded
template <int S, int TN>
__device__ __forceinline__ void beyond_sums(float (&sum)[S][TN], const h2 (&q)[S][TN / 2], const BeyondConst& w) {
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) {
            asm("v_fma_mix_f32 %0, %1, %2, %0 op_sel_hi:[1,0,0]" : "+v"(sum[i][2 * j]) : "v"(q[i][j]), "v"(w.kc));
            asm("v_fma_mix_f32 %0, %1, %2, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(sum[i][2 * j + 1]) : "v"(q[i][j]), "v"(w.kc));
        }
    __builtin_amdgcn_sched_barrier(0);
}
template <bool CLAMP, bool PRIO, int S, int TN>
__device__ __forceinline__ void beyond_round(float (&sum)[S][TN], const BeyondConst& w) {
    issue_last<PRIO>();
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) sum[i][j] = __uint_as_float(__float_as_uint(sum[i][j]) & w.mask);
    __builtin_amdgcn_sched_barrier(0);
    issue_first<PRIO>();
    if (CLAMP) {
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) sum[i][j] = med3(sum[i][j], w.nrof, w.rof);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// 32 steps, as rows_tile: operands are read a pair ahead, or four where a lone wave has few chains to wait with (LONE: there the next
// step's products stand between a sum and its mask)
template <int PM, int ORDER, bool CLAMP, bool LONE, int S, int TN, int BROW, int PITCH>
__device__ __forceinline__ void beyond_tile(float (&sum)[S][TN], float (&top)[S][TN], const uint32_t* arow, const uint32_t* Bs, const HalfConst& c,
                                            const BeyondConst& w) {
    constexpr int W = TN / 2, AHEAD = LONE ? 4 : 1, SLOTS = 2 * AHEAD, GROUP = LONE ? 8 : 4;
    constexpr bool PRIO = !LONE;
    uint32_t a[SLOTS][S], b0[SLOTS][W], b1[SLOTS][W];
    auto read = [&](int s, int k) {
#pragma unroll
        for (int i = 0; i < S; ++i) a[k][i] = arow[i * 8 * PITCH + s];
        read_words<W>(Bs + 2 * s * BROW, b0[k]);
        read_words<W>(Bs + (2 * s + 1) * BROW, b1[k]);
    };
    h2 q[2][S][W];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) read(s, s);
    issue_first<PRIO>();
    if (LONE) half_products<PM, false, S, TN, PRIO>(q[0], a[0], b0[0], c);
#pragma unroll 1
    for (int g = 0; g < 16; g += GROUP) {
#pragma unroll
        for (int u = 0; u < GROUP; ++u) {
            const int k = u % SLOTS, next = (u + 1) % SLOTS;
            read(u + AHEAD < GROUP ? g + u + AHEAD : min(g + u + AHEAD, 15), (u + AHEAD) % SLOTS);   // (the last ones again at the end)
            if (!LONE) half_products<PM, false, S, TN, PRIO>(q[0], a[k], b0[k], c);
            beyond_sums(sum, q[0], w);
            if (LONE) half_products<PM, true, S, TN, PRIO>(q[1], a[k], b1[k], c);
            beyond_round<CLAMP, PRIO>(sum, w);
            if (!LONE) half_products<PM, true, S, TN, PRIO>(q[1], a[k], b1[k], c);
            beyond_sums(sum, q[1], w);
            if (LONE) half_products<PM, false, S, TN, PRIO>(q[0], a[next], b0[next], c);
            beyond_round<CLAMP, PRIO>(sum, w);
        }
        if (ORDER == LBA_ORDER_CHUNK16 && (LONE || (g & 4))) {
#pragma unroll
            for (int i = 0; i < S; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) { top[i][j] += sum[i][j]; sum[i][j] = 0.0f; }
            __builtin_amdgcn_sched_barrier(0);
            beyond_round<CLAMP, PRIO>(top, w);
        }
    }
    issue_last<PRIO>();
}

// the steps of a list, as list_steps
template <int PM, bool CLAMP, int T, int U>
__device__ __forceinline__ void beyond_list(float (&sums)[T], const uint32_t* list, const char* Bb, int n, const HalfConst& c, const BeyondConst& w) {
    constexpr int W = T / 2;
    ListHead<U> h(list);
    uint32_t b[U][W];
    float sum[1][T];
#pragma unroll
    for (int j = 0; j < T; ++j) sum[0][j] = sums[j];
#pragma unroll
    for (int u = 0; u < U; ++u) read_words<W>(reinterpret_cast<const uint32_t*>(Bb + (h.e[u] >> 16)), b[u]);
    const uint32_t* const after = list + 2 * U;
    const auto round = [&](uint32_t (&e)[U], const uint32_t (&f)[U], int i) {
        h2 q[1][W];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t a1[1] = {e[u]};
            half_products<PM, false, 1, T, true>(q, a1, b[u], c);
            if (u == U - 1) ListHead<U>::read(after + i, e);
            read_words<W>(reinterpret_cast<const uint32_t*>(Bb + (f[u] >> 16)), b[u]);
            beyond_sums(sum, q, w);
            beyond_round<CLAMP, true>(sum, w);
        }
    };
    issue_first<true>();
    walk_list<U>(n, [&](int i) { round(h.e, h.f, i); }, [&](int i) { round(h.f, h.e, i); });
    issue_last<true>();
#pragma unroll
    for (int j = 0; j < T; ++j) sums[j] = sum[0][j];
}

// RANGE 0: every sum fits FP16 up to R_OF (half_carrier, lba_plan.cpp).  1, 2: R_OF lies beyond FP16's range; the bound that spares the
// clamp elsewhere shows that no sum leaves the range in the tile at hand (65504 in place of R_OF); a wave where it cannot goes on in FP32
// until its sums lie a whole tile inside the range again.  2: M = 10, FP16's own mantissa, which needs no mask.  M10E5 on 4096 x 4096 x 4096:
// 3220 us on FP32 carriers, 2070 here.
// EVENTS: the recompute call for the overflow plane alone (RANGE 0, no set of four rows): a part of a tile in which no sum can reach R_OF
// is the forward call's and its words are zero; any other runs half_bwd_tile.  A tile becomes lists only where the fixed bound covers it,
// since the steps a list leaves out have no event there (a saturated sum would repeat its own).
// ALONE: a wave has its SIMD to itself (lba_half_alone.hip): no turns, no lists, operands read further ahead.
template <int RW, int TN, int PM, int ORDER, int AMODE, int RANGE, bool EVENTS = false, bool ALONE = false>
__device__ __forceinline__ void rows_body(const KParams& p, uint32_t* __restrict__ smem, int m0, int n0) {
    using T = RowTile<RW, TN>;
    constexpr int BM = T::BM, BN = T::BN, S = T::SETS, W = TN / 2, U = T::U;
    constexpr bool HALF = T::HALF, MASK = RANGE != 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tx = lane & 7, g = lane >> 3;
    // staging: lane = 4 (row of the wave) + (piece of the row); B's pieces go to the lanes that have none of A's where that is possible
    const int ca = (lane >> 2) < RW ? (lane & 3) * BM + wave * RW + (lane >> 2) : -1;
    const int tidb = BN * 4 == 256 ? tid : (lane >= 32 && lane - 32 < BN ? wave * BN + lane - 32 : -1);
    const uint8_t* pA = p.A + (int64_t)blockIdx.z * p.stride_a;
    const uint8_t* pB = p.B + (int64_t)blockIdx.z * p.stride_b;
    float* pC = p.C + (int64_t)blockIdx.z * p.stride_c;
    static_assert(!EVENTS || (RANGE == 0 && !HALF), "the recompute call's tiles");

    set_flush_f32();
    set_round_zero_f16();
    set_flush_out_f16();
    if (RANGE != 0) set_round_zero();                          // of the FP32 sums; the bounds here have room for it

    HalfConst c;
    c.kc = as_h2(p.h_kc); c.rof = as_h2(p.h_rof); c.nrof = as_h2(p.h_rof ^ 0x80008000u); c.mask = p.h_mask_a; c.maskp = p.h_mask_p;
    asm volatile("" : "+v"(c.kc), "+v"(c.rof), "+v"(c.nrof), "+v"(c.mask), "+v"(c.maskp));

    h2 acc[S][W], top[S][W], acch[1][TN / 4 ? TN / 4 : 1], toph[1][TN / 4 ? TN / 4 : 1];
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j) { acc[i][j] = as_h2(0u); top[i][j] = as_h2(0u); }
#pragma unroll
    for (int j = 0; j < (TN / 4 ? TN / 4 : 1); ++j) { acch[0][j] = as_h2(0u); toph[0][j] = as_h2(0u); }

    uint32_t* const Aw = smem + 2 * T::B_WORDS + wave * RW * T::PITCH;     // the wave's rows of A
    const int ntiles = (p.K + HBK - 1) / HBK;
    __shared__ uint32_t half_norm[2][4];                       // per stage and wave: largest squared norm of a piece of A (low half), of B
    const bool dyn = half_follows_data(p);
    constexpr bool SMALL = S * TN <= 4, LONE = SMALL || ALONE, LISTS = ORDER == LBA_ORDER_SEQ && !LONE, PIECES = SMALL || AMODE >= 3;
    constexpr int AHEAD = LONE ? 4 : (S * TN >= 12 ? 1 : 2);   // pairs of steps whose operands are read ahead
    constexpr bool conv = AMODE == 2 || AMODE == 4;
    const RowPieces<BM> sa(pA, conv ? 1 : p.M, p.K, conv ? 0 : m0, ca);
    const RowPieces<BN> sb(pB, p.N, p.K, n0, tidb);
    ConvPieces sc = {};
    ConvLane cl = {};
    if (PIECES && conv) sc = ConvPieces::make<BM>(pA, p, m0, ca);
    if (!PIECES && AMODE == 2) cl = conv_lane<BM, HBK>(pA, p, m0, ca);
    constexpr int DEPTH = EVENTS ? 1 : AMODE == 4 && SMALL ? 2 : half_depth(S, TN);   // (two loads a piece: fewer tiles in flight)
    uint4 ra[DEPTH], rc[DEPTH], rb[DEPTH];
    const AlignedRow rowa(pA, conv ? 1 : p.M, p.K, conv ? 0 : m0 + ca % BM, ca >= 0 ? ca / BM * 16 : 0), rowb(pB, p.N, p.K, n0 + tidb % BN, tidb >= 0 ? tidb / BN * 16 : 0);
    auto fetch = [&](int t, int d) {
        const int k0 = tile_start(t);
        if (PIECES) {
            if (AMODE == 4)  load_piece(sc, p, k0, ra[d], rc[d]);
            else if (conv)   ra[d] = load_16(sc.first(p, k0)); // one tap
            else             ra[d] = load_piece(sa, k0);
            rb[d] = load_piece(sb, k0);
        } else {
            ra[d] = AMODE == 2 ? fetch_taps(cl, p, k0) : load_aligned(rowa, k0);
            rb[d] = load_aligned(rowb, k0);
        }
    };
    auto largest = [&]() {
        uint32_t mx = 0u;
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
            for (int j = 0; j < W; ++j)
                mx = pk_max_u16(mx, as_u32(ORDER == LBA_ORDER_CHUNK16 ? top[i][j] : acc[i][j]) & 0x7FFF7FFFu);
        if (HALF) {
#pragma unroll
            for (int j = 0; j < TN / 4; ++j)
                mx = pk_max_u16(mx, as_u32(ORDER == LBA_ORDER_CHUNK16 ? toph[0][j] : acch[0][j]) & 0x7FFF7FFFu);
        }
        return max_half(mx);
    };
    const HalfBound bound(p);
    int safe_tiles = 0;
    // the tile in LDS: steps of the two row sets' lists, and whether they are lists
    int n_first = 0, n_second = 0;
    bool listed = false;
    int wait = 0, pause = 0;                                   // tiles until zeros are counted again; that many after the next count in vain
    // Turns the wave's rows of the tile into lists if that saves enough; lane = code of the row.
    auto list_tile = [&](int t) -> bool {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint32_t x[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) x[r] = reinterpret_cast<const u16_any*>(Aw + r * T::PITCH)[lane];
        uint64_t nz[RW];
        int most[2] = {0, 0};
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            nz[r] = __ballot(x[r] != 0u);
            asm("s_max_u32 %0, %0, %1" : "+s"(most[r / 8]) : "s"(__builtin_popcountll(nz[r])) : "scc");
        }
        n_first = (most[0] + U - 1) & ~(U - 1);
        n_second = (most[1] + U - 1) & ~(U - 1);
        const int steps = p.K - t * HBK > 32 ? 64 : 32;
        const int dense = S == 2 ? 2 * steps : (HALF ? steps + steps / 2 : steps);
        // a step of a list takes 9/8 of an unrolled one, and building and starting the lists 12 to 14 of them (8192 x 512 x 2304 by the
        // share of zeros: 104 us for none left, 3.0 us per step and row set; unrolled 2.7)
        if ((HALF ? n_first + n_second / 2 : n_first + n_second) * 9 + 110 > dense * 8) return false;
        // A list runs with the clamp (or in FP32) unless the bound holds for all of its steps at once; where it does not but holds for the
        // 32 steps of an unrolled part, the parts most often run without, one after the other, and a clamped list takes half as long
        // again as one without (R_OF just above the sums, 50176 x 128 x 1152 behind a ReLU: 370 us with such lists, 263 so; 344
        // before there were lists)
        if (!EVENTS && !dyn && safe_tiles < 2) {
            const float mf = largest();
            safe_tiles = bound.safe(mf, nullptr);
            if (safe_tiles < 2) {
                if (bound.covers(mf, max(n_first, n_second))) safe_tiles = 2;
                else if (safe_tiles > 0) return false;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t row_of_b = (uint32_t)((t & 1) * T::B_WORDS * 4 + lane * T::BROW * 4) << 16;
        const uint32_t last = 63u - (uint32_t)lane;
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            // the non-zero codes in order, the zeros behind them from the end (all 64 words are written)
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(nz[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)nz[r], 0u));
            uint32_t slot;
            asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(slot) : "v"(at + last), "v"(at), "s"(nz[r]));
            Aw[r * T::PITCH + slot] = x[r] | row_of_b;
        }
        return true;
    };
    auto stage = [&](int t, int d) {
        uint4 va = ra[d];
        if (AMODE == 4 && SMALL) va = sc.codes(p, ra[d], rc[d], t * HBK);
        else if (AMODE == 4)     va = p.cv_vec ? sc.tap_codes(p, ra[d], t * HBK) : sc.row_codes(p, ra[d], rc[d], t * HBK);   // (filter rows shorter than a piece: the smallest grids alone)
        else if (PIECES && conv) va = sc.tap_codes(p, ra[d], t * HBK);
        else if (PIECES)         va = sa.codes(ra[d], t * HBK);
        uint4 vb = PIECES ? sb.codes(rb[d], t * HBK) : rb[d];
        if (!PIECES && (t + 1) * HBK > p.K) {                  // uniform: steps beyond K
            if (!conv) va = rowa.codes(va, t * HBK);
            vb = rowb.codes(vb, t * HBK);
        }
        const int st = t & 1;
        uint32_t wa[8], wb[8];
        decode_half(vb, p.h_shift_b, p.h_keep_b, p.h_scale_b, wb);
        store_half_b<BN>(smem + st * T::B_WORDS, tidb, wb);
        decode_half(va, p.h_shift_a, p.h_keep_a, p.h_scale_a, wa);
        if (ca >= 0) {
            uint4* const pairs = reinterpret_cast<uint4*>(Aw + (lane >> 2) * T::PITCH + (lane & 3) * 8);
            pairs[0] = make_uint4(wa[0], wa[1], wa[2], wa[3]);
            pairs[1] = make_uint4(wa[4], wa[5], wa[6], wa[7]);
        }
        listed = false;
        if (LISTS) {
            // worth counting: a zero among the first four codes of most pieces
            const uint32_t z = (va.x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu;
            const int hits = __builtin_popcountll(__ballot((z & 0x80808080u) != 0x80808080u && ca >= 0));
            if (EVENTS && safe_tiles < 2) safe_tiles = bound.safe(largest(), nullptr);
            if (wait > 0) {
                --wait;
            } else if (hits >= 4 * RW * 3 / 4 && (!EVENTS || safe_tiles >= 2)) {
                listed = list_tile(t);
                pause = listed ? 0 : min(2 * pause + 1, 15);
                wait = pause;
            }
        }
        if (dyn) {
            const uint32_t na = __float_as_uint(piece_norm2(wa)), nb = __float_as_uint(piece_norm2(wb));
            uint32_t m = ((na + 0xFFFFu) >> 16) | ((nb + 0xFFFFu) & 0xFFFF0000u);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m = pk_max_u16(m, (uint32_t)__shfl_xor((int)m, o, 64));
            if (lane == 0) half_norm[st][wave] = m;
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) fetch(d, d);               // (a tile beyond K reads codes inside the operands that nothing uses)
    if (LISTS && ca >= 0) pad_row<T>(lane & 3, [&](int w) { Aw[(lane >> 2) * T::PITCH + w] = 0u; });
    stage(0, 0);
    if (DEPTH > 1) fetch(DEPTH, 0);
    __syncthreads();

    int base = 0, beyond = -1, from = 0;                       // the tile a packed stretch starts at; the tile and its part where it ends
    // a lane's words of its rows (one per chain) as word `word` of a plane; non-temporal, see store_event_words
    uint32_t of2[S][TN] = {};
    auto store_words = [&](uint32_t* plane, int word, const uint32_t (&w)[S][TN]) {
        if (!plane) return;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int m = m0 + wave * RW + 8 * i + g, n = n0 + tx * TN;
            if (m >= p.M) continue;
            uint32_t* dst = plane + ((int64_t)word * p.M + m) * p.N + n;
            if (p.c_vec && n + TN - 1 < p.N) {
#pragma unroll
                for (int j = 0; j + 3 < TN; j += 4)
                    __builtin_nontemporal_store(u32x4_any{w[i][j], w[i][j + 1], w[i][j + 2], w[i][j + 3]}, reinterpret_cast<u32x4_any*>(dst + j));
            } else {
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (n + j < p.N) __builtin_nontemporal_store(w[i][j], dst + j);
            }
        }
    };
    // the wave's words where nothing overflows: whole rows by a store, 16 bytes a lane (a lane's own eight words in two stores with gaps
    // between them went to memory as partial lines: 3985 x 770 x 771 in chunks 300 us instead of 170)
    auto store_no_events = [&](int word) {
        constexpr int LANES = BN / 4, ROWS = 64 / LANES;
        if (!p.of_mask) return;
        int l = lane;
        if (!ALONE) asm volatile("" : "+v"(l));              // addresses made here, not kept in registers over the loop
#pragma unroll
        for (int i = 0; i < RW; i += ROWS) {
            const int m = m0 + wave * RW + i + l / LANES, n = n0 + l % LANES * 4;
            if (m >= p.M) continue;
            uint32_t* dst = p.of_mask + ((int64_t)word * p.M + m) * p.N + n;
            if (p.c_vec && n + 3 < p.N) {
                __builtin_nontemporal_store(u32x4_any{0u, 0u, 0u, 0u}, reinterpret_cast<u32x4_any*>(dst));
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (n + j < p.N) __builtin_nontemporal_store(0u, dst + j);
            }
        }
    };
    const uint32_t* const arow = Aw + g * T::PITCH;
    const uint32_t* const arowh = Aw + (8 + (lane >> 4)) * T::PITCH;       // the 4-row set: 16 lanes a row
    // C = S * 2^out_exp, zero written as +0
    auto store = [&](int m, int n, auto sum, auto count) {
        constexpr int CT = decltype(count)::value;
        if (m >= p.M) return;
        float v[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) v[j] = __builtin_ldexpf(sum(j), p.out_exp - 112) + 0.0f;    // -0 + 0 is +0
        float* dst = pC + (int64_t)m * p.N + n;
        if (CT % 4 == 0 && p.c_vec && n + CT - 1 < p.N) {
#pragma unroll
            for (int j = 0; j + 3 < CT; j += 4) *reinterpret_cast<f32x4_any*>(dst + j) = f32x4_any{v[j], v[j + 1], v[j + 2], v[j + 3]};
        } else if (CT == 2 && p.c_vec && n + 1 < p.N) {
            *reinterpret_cast<f32x2_any*>(dst) = f32x2_any{v[0], v[CT - 1]};
        } else {
#pragma unroll
            for (int j = 0; j < CT; ++j)
                if (n + j < p.N) dst[j] = v[j];
        }
    };
    const int row0 = m0 + wave * RW + g, rowh = m0 + wave * RW + 8 + (lane >> 4);
    const int col0 = n0 + tx * TN, colh = n0 + (lane & 15) * (TN / 2);
    for (;;) {
        for (int t0 = base; t0 < ntiles; t0 += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const int t = t0 + d;
                if (t >= ntiles) break;
                const bool more = (t + 1) < ntiles;
                if (DEPTH == 1) fetch(t + 1, 0);
                const int parts = p.K - t * HBK > 32 ? 2 : 1;      // steps beyond K are products of zeros: skipped 32 at a time
                if (LISTS && listed) {
                    if (safe_tiles < parts && dyn) {
                        const float mf = largest();
                        safe_tiles = bound.safe(mf, nullptr);
                        if (safe_tiles < parts) safe_tiles = bound.follows(mf, half_norm[t & 1], parts) ? parts : 0;
                    }
                    const char* const Bb = reinterpret_cast<const char*>(smem + tx * W);
                    const char* const Bh = reinterpret_cast<const char*>(smem + (lane & 15) * (W / 2));
                    if constexpr (EVENTS) {
                        for (int part = 0; part < parts; ++part) store_no_events(2 * t + part);
                    }
                    ListHead<U> h0(arow), h1(HALF ? arowh : arow + (S == 2 ? 8 * T::PITCH : 0));
                    if (safe_tiles >= parts) {
                        safe_tiles -= parts;
                        list_steps<PM, false, MASK, TN, U>(acc[0], h0, arow, Bb, n_first, c);
                        if constexpr (S == 2) list_steps<PM, false, MASK, TN, U>(acc[1], h1, arow + 8 * T::PITCH, Bb, n_second, c);
                        if constexpr (HALF) list_steps<PM, false, MASK, TN / 2, U>(acch[0], h1, arowh, Bh, n_second, c);
                    } else if constexpr (RANGE != 0) {
                        beyond = t;
                        break;
                    } else {
                        safe_tiles = 0;
                        list_steps<PM, true, MASK, TN, U>(acc[0], h0, arow, Bb, n_first, c);
                        if constexpr (S == 2) list_steps<PM, true, MASK, TN, U>(acc[1], h1, arow + 8 * T::PITCH, Bb, n_second, c);
                        if constexpr (HALF) list_steps<PM, true, MASK, TN / 2, U>(acch[0], h1, arowh, Bh, n_second, c);
                    }
                } else {
                    for (int part = 0; part < parts; ++part) {
                        const uint32_t* const Bp = smem + (t & 1) * T::B_WORDS + part * 32 * T::BROW;
                        const uint32_t* const Bs = Bp + tx * W;
                        const uint32_t* const Bh = Bp + (lane & 15) * (W / 2);
                        if (safe_tiles == 0) safe_tiles = bound.safe(largest(), dyn ? half_norm[t & 1] : nullptr);
                        const int word = 2 * t + part;             // of the planes
                        if (safe_tiles > 0) {
                            --safe_tiles;
                            if constexpr (EVENTS) store_no_events(word);
                            rows_tile<PM, ORDER, false, MASK, LONE, AHEAD, S, TN, T::BROW, T::PITCH>(acc, top, arow + part * 16, Bs, c);
                            if constexpr (HALF) rows_tile<PM, ORDER, false, MASK, ALONE, ALONE ? 4 : (TN / 2 >= 8 ? 2 : 4), 1, TN / 2, T::BROW, T::PITCH>(acch, toph, arowh + part * 16, Bh, c);
                        } else if constexpr (EVENTS) {
                            const HalfBwdConst cb(p);
                            uint32_t of[S][TN], none[S][TN], none2[S][TN];
#pragma unroll
                            for (int i = 0; i < S; ++i)
#pragma unroll
                                for (int j = 0; j < TN; ++j) { of[i][j] = 0u; none[i][j] = 0u; none2[i][j] = 0u; }
                            half_bwd_tile<PM, ORDER, false, false, S, TN, !LONE>(acc, top, of, none, of2, none2, 2 * (word & 15),
                                [&](int k, uint32_t (&a)[S]) {
#pragma unroll
                                    for (int i = 0; i < S; ++i) a[i] = arow[i * 8 * T::PITCH + part * 16 + k];
                                },
                                [&](int k, uint32_t (&b)[W]) { read_words<W>(Bs + k * T::BROW, b); }, cb);
                            const int valid = p.K - 32 * word;     // a saturated sum stays at R_OF beyond K
                            if (valid < 32) {
#pragma unroll
                                for (int i = 0; i < S; ++i)
#pragma unroll
                                    for (int j = 0; j < TN; ++j) of[i][j] &= (1u << valid) - 1u;
                            }
                            if (ORDER == LBA_ORDER_SEQ && p.map_dx) mark_bricks_of_rows<RW, TN>(of, m0, n0, word, p);
                            store_words(p.of_mask, word, of);
                        } else if constexpr (RANGE != 0) {
                            beyond = t;
                            from = part;
                            break;
                        } else {
                            rows_tile<PM, ORDER, true, MASK, LONE, AHEAD, S, TN, T::BROW, T::PITCH>(acc, top, arow + part * 16, Bs, c);
                            if constexpr (HALF) rows_tile<PM, ORDER, true, MASK, ALONE, ALONE ? 4 : (TN / 2 >= 8 ? 2 : 4), 1, TN / 2, T::BROW, T::PITCH>(acch, toph, arowh + part * 16, Bh, c);
                        }
                    }
                    if (RANGE != 0 && beyond >= 0) break;
                }
                if constexpr (EVENTS && ORDER == LBA_ORDER_CHUNK16) {
                    // two chunks a word of the plane: a second-level word is complete after 16 of them
                    const int word = 2 * t + parts - 1;
                    if ((word & 15) == 15 || t + 1 == ntiles) {
                        const int left = ((p.K + 15) >> 4) - 32 * (word >> 4);
                        const uint32_t vmask = left >= 32 ? 0xFFFFFFFFu : (1u << left) - 1u;
#pragma unroll
                        for (int i = 0; i < S; ++i)
#pragma unroll
                            for (int j = 0; j < TN; ++j) of2[i][j] &= vmask;
                        if (p.of_mask2) store_words(p.of_mask2, word >> 4, of2);
#pragma unroll
                        for (int i = 0; i < S; ++i)
#pragma unroll
                            for (int j = 0; j < TN; ++j) of2[i][j] = 0u;
                    }
                }
                if (more) {
                    constexpr int next = (DEPTH > 1) ? 1 : 0;
                    stage(t + 1, (d + next) % DEPTH);
                    if (DEPTH > 1) fetch(t + 1 + DEPTH, (d + next) % DEPTH);
                }
                __syncthreads();
            }
            if (RANGE != 0 && beyond >= 0) break;
        }

        if constexpr (RANGE == 0) {
            break;
        } else {
            if (beyond < 0) break;
            // a stretch in FP32
            constexpr int HT = HALF ? TN / 2 : 2;
            const BeyondConst w(p);
            float sum[S][TN], tops[S][TN], sumh[1][HT], toph2[1][HT];
            auto wide = [](const h2* s, int j) { return (float)(j & 1 ? s[j / 2].y : s[j / 2].x) * 0x1p-112f; };
#pragma unroll
            for (int i = 0; i < S; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) { sum[i][j] = wide(acc[i], j); tops[i][j] = wide(top[i], j); }
            if constexpr (HALF) {
#pragma unroll
                for (int j = 0; j < HT; ++j) { sumh[0][j] = wide(acch[0], j); toph2[0][j] = wide(toph[0], j); }
            }
            auto most = [&]() {
                float m = 0.0f;
#pragma unroll
                for (int i = 0; i < S; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) m = __builtin_fmaxf(m, __builtin_fabsf(ORDER == LBA_ORDER_CHUNK16 ? tops[i][j] : sum[i][j]));
                if constexpr (HALF) {
#pragma unroll
                    for (int j = 0; j < HT; ++j) m = __builtin_fmaxf(m, __builtin_fabsf(ORDER == LBA_ORDER_CHUNK16 ? toph2[0][j] : sumh[0][j]));
                }
                return m;
            };
            int t = beyond, quiet = 0;                             // parts in which no sum reaches R_OF
            float mx = most();
            for (;;) {
                if (AMODE != 4) fetch(t + 1, 0);               // (two loads a piece would cost the packed stretch its registers)
                const int parts = p.K - t * HBK > 32 ? 2 : 1;
                if (LISTS && listed) {
                    const char* const Bb = reinterpret_cast<const char*>(smem + tx * W);
                    const char* const Bh = reinterpret_cast<const char*>(smem + (lane & 15) * (W / 2));
                    const auto lists = [&](auto clamp) {
                        constexpr bool CLAMP = decltype(clamp)::value != 0;
                        beyond_list<PM, CLAMP, TN, U>(sum[0], arow, Bb, n_first, c, w);
                        if constexpr (S == 2) beyond_list<PM, CLAMP, TN, U>(sum[1], arow + 8 * T::PITCH, Bb, n_second, c, w);
                        if constexpr (HALF) beyond_list<PM, CLAMP, TN / 2, U>(sumh[0], arowh, Bh, n_second, c, w);
                    };
                    if (quiet < parts && __all(mx < p.fast_thresh4)) quiet = 4;
                    if (quiet >= parts) { quiet -= parts; lists(IntConst<0>{}); }
                    else                { quiet = 0; lists(IntConst<1>{}); }
                    mx = most();
                } else {
                    for (int part = from; part < parts; ++part) {
                        const uint32_t* const Bp = smem + (t & 1) * T::B_WORDS + part * 32 * T::BROW;
                        const uint32_t* const Bs = Bp + tx * W;
                        const uint32_t* const Bh = Bp + (lane & 15) * (W / 2);
                        const auto tile = [&](auto clamp) {
                            constexpr bool CLAMP = decltype(clamp)::value != 0;
                            beyond_tile<PM, ORDER, CLAMP, SMALL, S, TN, T::BROW, T::PITCH>(sum, tops, arow + part * 16, Bs, c, w);
                            if constexpr (HALF) beyond_tile<PM, ORDER, CLAMP, false, 1, TN / 2, T::BROW, T::PITCH>(sumh, toph2, arowh + part * 16, Bh, c, w);
                        };
                        if (quiet == 0) quiet = __all(mx < p.fast_thresh4) ? 4 : (__all(mx < p.fast_thresh) ? 1 : 0);
                        if (quiet > 0) { --quiet; tile(IntConst<0>{}); }
                        else           tile(IntConst<1>{});
                        mx = most();
                    }
                }
                from = 0;
                const bool more = t + 1 < ntiles;
                if (AMODE == 4) fetch(t + 1, 0);
                if (more) stage(t + 1, 0);
                __syncthreads();                                   // (one a tile, as in the packed stretch of other waves)
                ++t;
                if (!more) {
#pragma unroll
                    for (int i = 0; i < S; ++i) store(row0 + 8 * i, col0, [&](int j) { return (ORDER == LBA_ORDER_CHUNK16 ? tops[i][j] : sum[i][j]) * 0x1p112f; }, IntConst<TN>{});
                    if constexpr (HALF) store(rowh, colh, [&](int j) { return (ORDER == LBA_ORDER_CHUNK16 ? toph2[0][j] : sumh[0][j]) * 0x1p112f; }, IntConst<TN / 2>{});
                    return;
                }
                safe_tiles = bound.safe(mx * 0x1p112f, nullptr);
                if (safe_tiles >= 2) break;
            }
            // back: every sum is inside FP16's range and has at most 11 bits, at 2^-14 or above
            auto narrow = [](float x, float y) { return __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(x * 0x1p112f, y * 0x1p112f)); };
#pragma unroll
            for (int i = 0; i < S; ++i)
#pragma unroll
                for (int j = 0; j < W; ++j) { acc[i][j] = narrow(sum[i][2 * j], sum[i][2 * j + 1]); top[i][j] = narrow(tops[i][2 * j], tops[i][2 * j + 1]); }
            if constexpr (HALF) {
#pragma unroll
                for (int j = 0; j < HT / 2; ++j) { acch[0][j] = narrow(sumh[0][2 * j], sumh[0][2 * j + 1]); toph[0][j] = narrow(toph2[0][2 * j], toph2[0][2 * j + 1]); }
            }
            base = t;
            beyond = -1;
            if (DEPTH > 1) {                                       // the tiles ahead, in the slots the loop expects them in
#pragma unroll
                for (int d = 1; d <= DEPTH; ++d) fetch(base + d, d % DEPTH);
            }
        }
    }

    if (EVENTS && !p.C) return;
    auto value = [](const h2* s, int j) { return (float)(j & 1 ? s[j / 2].y : s[j / 2].x); };
#pragma unroll
    for (int i = 0; i < S; ++i) store(row0 + 8 * i, col0, [&](int j) { return value(ORDER == LBA_ORDER_CHUNK16 ? top[i] : acc[i], j); }, IntConst<TN>{});
    if constexpr (HALF) store(rowh, colh, [&](int j) { return value(ORDER == LBA_ORDER_CHUNK16 ? toph[0] : acch[0], j); }, IntConst<TN / 2>{});
}

// The smallest grids, at most one or two workgroups per CU: four waves run the chains of a 32 x BN tile (8 rows each, BN / 8 columns
// per lane) and four others fetch and decode the k-tile after it.  What bounds such a call is one wave's issue, 4 cycles an instruction and
// 12 a step (multiply-add, next product, mask), so everything else leaves that wave: staging, most LDS reads (B lies in groups of steps, one
// 16-byte read for four or two of them, 8 cycles each among other instructions), and branches: a taken one costs a lone wave 40 to 130
// cycles (measured with loops of 16 to 256 steps).  So a tile of 64 steps is run straight through, its operands read ahead across its
// end, and a loop has one branch a tile.  Lists of non-zero codes do not pay here: a step then needs a read and an address of its own.
// Four waves that do both -> parts of 32 steps that start anew -> here, us: 64 x 1000 x 2048 44 -> 26.9 -> 22.4, 300 x 300 x 1500 36 -> 20.2 ->
// 16.7, 512 x 512 x 512 16 -> 12.6 -> 11.4, 416 x 480 x 3312 64.6 -> 57.2 for the last two, with R_OF near the sums (clamped) 300 x 300 x 1500
// 29 -> 22.
template <int TN>
struct StagedTile {
    static constexpr int BM = 32, BN = 8 * TN, W = TN / 2, GROUP = 4 / W;  // steps of B in 16 bytes
    static constexpr int B16 = 16 * BN / 2 + 16;                           // words of 16 steps of B, and a shift of their banks for the lanes that write them
    static constexpr int B_WORDS = HBK / 16 * B16, PAIRS = HBK / 2 + 4;    // a row's words (k, k + 1), and a shift of its banks
    static constexpr int STAGE = B_WORDS + BM * PAIRS, STAGES = 4, WORDS = STAGES * STAGE;
};

// The 16 codes of a column's piece in that layout, [k / GROUP][lane of 8][k % GROUP][word], as half words: the lane has nothing else to
// wait for, and the pairs of columns need no exchange between lanes.
template <int TN>
__device__ __forceinline__ void store_staged_b(uint32_t* __restrict__ dst, int col, int kq, const uint32_t (&w)[8]) {
    using T = StagedTile<TN>;
    u16_any* const to = reinterpret_cast<u16_any*>(dst + kq * T::B16) + col / TN * 8 + col % TN;
#pragma unroll
    for (int j = 0; j < 16; ++j) to[(j / T::GROUP * 8 * T::GROUP + j % T::GROUP) * TN] = (uint16_t)(w[j / 2] >> (j & 1 ? 16 : 0));
}

// The operands of a lane's chains ahead of the steps: quads of A's words (eight steps each) and of B's (GROUP steps each), and the
// products of the step to come.
template <int TN>
struct StagedAhead {
    using T = StagedTile<TN>;
    static constexpr int W = T::W, G = T::GROUP, STEPS = TN == 2 ? 16 : 8, AQ = STEPS / 8 * 2, BQ = STEPS / G * 2;
    uint32_t a[AQ][4], b[BQ][4];
    h2 q[1][W];
    // quads i of the tile at a base
    __device__ __forceinline__ void read_a(const uint32_t* base, int i) { read_words<4>(base + 4 * i, a[i % AQ]); }
    __device__ __forceinline__ void read_b(const uint32_t* base, int i) { read_words<4>(base + i / (16 / G) * T::B16 + i % (16 / G) * 32, b[i % BQ]); }
    // the words of step k: A's, whose half is k & 1, and B's
    __device__ __forceinline__ uint32_t word_a(int k) const { return a[k / 8 % AQ][k / 2 % 4]; }
    template <int PM>
    __device__ __forceinline__ void product(int k, const HalfConst& c) {
        const uint32_t x[1] = {word_a(k)};
        uint32_t y[W];
#pragma unroll
        for (int j = 0; j < W; ++j) y[j] = b[k / G % BQ][k % G * W + j];
        if (k & 1) half_products<PM, true, 1, TN, false>(q, x, y, c);
        else       half_products<PM, false, 1, TN, false>(q, x, y, c);
    }
};

// Steps FROM to FROM + 31 of a tile whose operands are at (ab, Bb), the next tile's at (an, Bn).  Operands are read STEPS steps ahead, across
// the end of the tile, and products are taken before the sum ahead of them is rounded: a tile starts with everything it needs in
// registers.
template <int PM, int ORDER, bool CLAMP, int TN, int FROM>
__device__ __forceinline__ void staged_steps(h2 (&sum)[1][TN / 2], h2 (&top)[1][TN / 2], StagedAhead<TN>& o, const uint32_t* ab, const uint32_t* Bb, const uint32_t* an,
                                             const uint32_t* Bn, const HalfConst& c) {
    using S = StagedAhead<TN>;
    constexpr int W = S::W, G = S::G, AHEAD = S::STEPS;
#pragma unroll
    for (int k = FROM; k < FROM + 32; ++k) {
        if (k % 8 == 0 || k % G == 0) asm volatile("" ::: "memory");   // (reads stay where they are)
        if (k % 8 == 0) {
            const int i = (k + AHEAD) / 8;
            if (i < HBK / 8) o.read_a(ab, i);
            else             o.read_a(an, i - HBK / 8);
        }
        if (k % G == 0) {
            const int i = (k + AHEAD) / G;
            if (i < HBK / G) o.read_b(Bb, i);
            else             o.read_b(Bn, i - HBK / G);
        }
        const uint32_t x[1] = {o.word_a(k)};
        uint32_t y[W];
#pragma unroll
        for (int j = 0; j < W; ++j) y[j] = o.b[k / G % S::BQ][k % G * W + j];
        if (k & 1) half_sums<PM, true, 1, TN>(sum, o.q, x, y, c);
        else       half_sums<PM, false, 1, TN>(sum, o.q, x, y, c);
        o.template product<PM>((k + 1) % HBK, c);
        half_round<CLAMP, 1, TN, false>(sum, c);
        if (ORDER == LBA_ORDER_CHUNK16 && k % 16 == 15) half_level2<CLAMP, 1, TN>(top, sum, c);
    }
}

template <int TN, int PM, int CONV, int ORDER>
__device__ __forceinline__ void staged_body(const KParams& p, uint32_t* __restrict__ smem, int m0, int n0) {
    using T = StagedTile<TN>;
    constexpr int W = TN / 2, AHEAD = kTilesAhead;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
    const bool stager = __builtin_amdgcn_readfirstlane(tid >> 8) != 0;
    const uint8_t* pA = p.A + (int64_t)blockIdx.z * p.stride_a;
    const uint8_t* pB = p.B + (int64_t)blockIdx.z * p.stride_b;
    __shared__ uint32_t half_norm[4][4];                       // of tiles t & 3 (the tile ahead and one being staged beside the tile read)
    const bool dyn = half_follows_data(p);
    const int ntiles = (p.K + HBK - 1) / HBK;
    set_flush_f32();
    set_round_zero_f16();
    set_flush_out_f16();

    // A barrier in front of the first tile, which is staged then, and one in the middle of every tile: the next one is staged, and the
    // stage of the one before is no longer read.
    if (stager) {
        // waves 0 and 1: 16 rows of A each, four lanes a row; the others: 16 columns of B each (with TN = 2 the last has none)
        const bool isb = wave >= 2;                            // uniform, as all that follows from it
        const int line = (wave & 1) * 16 + (lane >> 2), kq = lane & 3;
        const bool mine = !isb || line < T::BN;
        int rows_a = CONV ? 1 : p.M, rows_b = p.N;
        asm("" : "+s"(rows_a), "+s"(rows_b));                  // (two neighbours in p and a choice of them went through scratch memory)
        const RowPieces<32> s(isb ? pB : pA, isb ? rows_b : rows_a, p.K, isb ? n0 : (CONV ? 0 : m0), mine && (isb || !CONV) ? kq * 32 + line : -1);
        ConvPieces sc = {};
        if (CONV && !isb) sc = ConvPieces::make<T::BM>(pA, p, m0, kq * 32 + line);
        const int shift = isb ? p.h_shift_b : p.h_shift_a;
        const uint32_t keep = isb ? p.h_keep_b : p.h_keep_a, scale = isb ? p.h_scale_b : p.h_scale_a;
        uint4 r[AHEAD], r2[CONV == 2 ? AHEAD : 1];
        auto fetch = [&](int t, int d) {                       // (a tile beyond K reads codes inside the operands that nothing uses)
            const int k0 = tile_start(t);
            if (CONV) {
                const uint8_t* a = s.address(k0);
                if (!isb) a = sc.first(p, k0);
                r[d] = load_16(a);
                if constexpr (CONV == 2) {
                    if (!isb) a = sc.second(p, k0);
                    r2[d] = load_16(a);
                }
            } else {
                r[d] = load_piece(s, k0);
            }
        };
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) fetch(d, d);
        static_assert(AHEAD == T::STAGES, "a tile's stage is its slot of the loads in flight");
        for (int t0 = 0; t0 < ntiles; t0 += AHEAD) {
#pragma unroll
            for (int d = 0; d < AHEAD; ++d) {
                const int t = t0 + d;
                if (t >= ntiles) break;
                uint32_t* const st = smem + d * T::STAGE;
                uint4 v = r[d];
                if (!CONV || isb)             v = s.codes(v, t * HBK);
                else if constexpr (CONV == 2) v = sc.row_codes(p, v, r2[d], t * HBK);
                else                          v = sc.tap_codes(p, v, t * HBK);
                uint32_t w[8];
                decode_half(v, shift, keep, scale, w);
                if (isb) {
                    if (mine) store_staged_b<TN>(st, line, kq, w);
                } else {
                    uint4* const pairs = reinterpret_cast<uint4*>(st + T::B_WORDS + line * T::PAIRS + kq * 8);
                    pairs[0] = make_uint4(w[0], w[1], w[2], w[3]);
                    pairs[1] = make_uint4(w[4], w[5], w[6], w[7]);
                }
                if (dyn) {
                    const uint32_t n2 = wave_max_u16((__float_as_uint(piece_norm2(w)) + 0xFFFFu) >> 16);
                    if (lane == 63) half_norm[t & 3][wave] = isb ? n2 << 16 : n2;
                }
                fetch(t + AHEAD, d);
                __syncthreads();
            }
        }
        __syncthreads();
        return;
    }

    HalfConst c;
    c.kc = as_h2(p.h_kc); c.rof = as_h2(p.h_rof); c.nrof = as_h2(p.h_rof ^ 0x80008000u); c.mask = p.h_mask_a; c.maskp = p.h_mask_p;
    asm volatile("" : "+v"(c.kc), "+v"(c.rof), "+v"(c.nrof), "+v"(c.mask), "+v"(c.maskp));
    h2 acc[1][W], top[1][W];
#pragma unroll
    for (int j = 0; j < W; ++j) { acc[0][j] = as_h2(0u); top[0][j] = as_h2(0u); }
    const h2 (&kept)[1][W] = ORDER == LBA_ORDER_CHUNK16 ? top : acc;
    const int tx = lane & 7, g = lane >> 3;
    const HalfBound bound(p);
    __builtin_amdgcn_s_setprio(3);                             // the chain is what everything waits for
    const uint32_t* const Bl = smem + tx * 4;
    const uint32_t* const al = smem + T::B_WORDS + (wave * 8 + g) * T::PAIRS;
    StagedAhead<TN> o;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < StagedAhead<TN>::STEPS / 8; ++i) o.read_a(al, i);
#pragma unroll
    for (int i = 0; i < StagedAhead<TN>::STEPS / T::GROUP; ++i) o.read_b(Bl, i);
    o.template product<PM>(0, c);
    const auto largest = [&]() {
        uint32_t mx = 0u;
#pragma unroll
        for (int j = 0; j < W; ++j) mx = pk_max_u16(mx, as_u32(kept[0][j]) & 0x7FFF7FFFu);
        return max_half(mx);
    };
    // n tiles.  A loop for each form, straight through a tile: a taken branch costs a lone wave 40 to 130 cycles (three or four of them for every
    // 32 steps were as much again as the steps), an instruction 4.
    const bool half = ((p.K - 1) & 32) == 0;                   // the last tile's second half lies beyond K (other steps there are products of zeros)
    int t = 0;                                                 // the tile to come
    const auto tiles = [&](auto clamp, int n) {
#pragma unroll 1
        for (n = min(n, ntiles - t); n > 0; --n) {
            const int at = (t & 3) * T::STAGE, then = (++t & 3) * T::STAGE;
            staged_steps<PM, ORDER, decltype(clamp)::value != 0, TN, 0>(acc, top, o, al + at, Bl + at, al + then, Bl + then, c);
            __syncthreads();
            if (t == ntiles && half) break;
            staged_steps<PM, ORDER, decltype(clamp)::value != 0, TN, 32>(acc, top, o, al + at, Bl + at, al + then, Bl + then, c);
        }
    };
    while (t < ntiles) {
        const float mf = largest();
        const int safe = bound.safe(mf, nullptr);
        if (safe >= 2)                                                    tiles(IntConst<0>{}, safe / 2);
        else if (dyn && bound.follows(mf, half_norm[t & 3], 2))           tiles(IntConst<0>{}, 1);
        else                                                              tiles(IntConst<1>{}, dyn ? 1 : 2);
    }
    const int m = m0 + wave * 8 + g, n = n0 + tx * TN;
    if (m >= p.M) return;
    float* const dst = p.C + (int64_t)blockIdx.z * p.stride_c + (int64_t)m * p.N + n;
    float v[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) v[j] = __builtin_ldexpf((float)(j & 1 ? kept[0][j / 2].y : kept[0][j / 2].x), p.out_exp - 112) + 0.0f;   // -0 + 0 is +0
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

template <int TN, int PM, int CONV, int ORDER>
__device__ __forceinline__ void staged_grid(const KParams& p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[StagedTile<TN>::WORDS];
    const int by = TN == 2 ? blockIdx.x / p.mix_gx_tail : blockIdx.y, bx = TN == 2 ? blockIdx.x - by * p.mix_gx_tail : blockIdx.x;
    staged_body<TN, PM, CONV, ORDER>(p, smem, bx * 32, by * 8 * TN);
}
// 512 lanes.  Row-major operands of any alignment; im2col rows, CONV 1: pieces are channels of one tap (cv_vec), 2: pieces
// span at most two filter rows.  One kernel for both waited for its loads where the branch around the second one met (3 x 3 on 56 x 56 x
// 64 29.6 us, 17.5 so).  lba_half_kernel -> here, one image: 7 x 7 x 512 to 512 channels, 3 x 3, 155 -> 84 us, 14 x 14 x 256 81 -> 45, 28 x
// 28 x 128 42 -> 24, 56 x 56 x 64 25.3 -> 17.6, a stem (112 x 112 x 3, 7 x 7) 12.6 -> 10.5; 8 of 7 x 7 x 512 177 -> 113 (since tiles are run
// straight through another 5 to 23 % less, the stem as before).  Products that Q_prod truncates and the chunked order, 256-lane workgroups of 32 x 32 or 64 x 64
// -> here: 350 x 350 x 700 M4E3 27.9 -> 13.7 us, chunked 28.4 -> 14.2, E4M3 with 5-bit products 55.7 -> 11.9; 700 x 500 x 500 31.7 -> 21.6; chunked 3 x 3 on
// 14 x 14 x 256 50.0 -> 27.6, 8 of 7 x 7 x 512 125 -> 81; a batch of 60 64 x 64 x 256 11.8 -> 7.9.
template <int TN, int PM, int ORDER>
__global__ void __launch_bounds__(512, 4) lba_half_staged_kernel(const KParams p) { staged_grid<TN, PM, 0, ORDER>(p); }
template <int TN, int PM, int CONV, int ORDER>
__global__ void __launch_bounds__(512, 4) lba_half_staged_conv_kernel(const KParams p) { staged_grid<TN, PM, CONV, ORDER>(p); }

template <int TM, int TN, int PM, int ORDER, int AMODE, int RANGE>
__device__ __forceinline__ void rows_plain(const KParams& p) {
    constexpr int RW = TM == 4 ? 16 : 8, TR = TN == 4 ? 8 : 4;
    __shared__ __attribute__((aligned(16))) uint32_t smem[RowTile<RW, TR>::WORDS];
    rows_body<RW, TR, PM, ORDER, AMODE, RANGE>(p, smem, blockIdx.x * 16 * TM, blockIdx.y * 16 * TN);
}
template <int PM, int ORDER, int AMODE, int RANGE, bool ALONE = false>
__device__ __forceinline__ void rows_mixed(const KParams& p) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[RowTile<16, 8>::WORDS];
    const int b = blockIdx.x;
    if (b < p.mix_main) {                                      // uniform
        const int by = b / p.mix_gx_main, bx = b - by * p.mix_gx_main;
        rows_body<16, 8, PM, ORDER, AMODE, RANGE, false, ALONE>(p, smem, bx * 64, by * 64);
    } else if (b < p.mix_main + p.mix_half) {
        const int t = b - p.mix_main;
        const int by = t / p.mix_gx_half, bx = t - by * p.mix_gx_half;
        rows_body<12, 8, PM, ORDER, AMODE, RANGE, false, ALONE>(p, smem, p.mix_m_main + bx * 48, by * 64);
    } else {
        const int t = b - p.mix_main - p.mix_half;
        const int by = t / p.mix_gx_tail, bx = t - by * p.mix_gx_tail;
        if (p.mix_tail16) rows_body<8, 2, PM, ORDER, AMODE, RANGE>(p, smem, p.mix_m_half + bx * 32, by * 16);   // uniform
        else              rows_body<8, 4, PM, ORDER, AMODE, RANGE>(p, smem, p.mix_m_half + bx * 32, by * 32);
    }
}

// The grids of lba_fast_kernel and lba_fast_mixed_kernel (the same tiles, numbered the same) on packed carriers: 16 TM x 16 TN outputs.
// AMODE 0: row-major, 16-byte rows; 3: row-major, any K and alignment; 2: im2col rows, C % 16 == 0 and 16-byte rows; 4: any other.
template <int TM, int TN, int PM, int ORDER, int AMODE>
__global__ void __launch_bounds__(256, LBA_FAST_MIN_WAVES) lba_half_kernel(const KParams p) { rows_plain<TM, TN, PM, ORDER, AMODE, 0>(p); }
template <int PM, int ORDER, int AMODE>
__global__ void __launch_bounds__(256, LBA_FAST_MIN_WAVES) lba_half_mixed_kernel(const KParams p) { rows_mixed<PM, ORDER, AMODE, 0>(p); }

// Accumulators whose R_OF lies beyond FP16's range (RANGE 1, 2).  (im2col rows of any channel count: with a fourth wave per SIMD the two forms of
// the tile spill on the square lane blocks, 37 x 225 x 226 x 3, 7 x 7: 223 us, 200 so; the others are
// faster with it)
template <int TM, int TN, int ORDER, int AMODE, int RANGE>
__global__ void __launch_bounds__(256, AMODE == 4 && TM == TN ? 3 : LBA_FAST_MIN_WAVES) lba_wide_kernel(const KParams p) { rows_plain<TM, TN, PM_FLUSH, ORDER, AMODE, RANGE>(p); }
template <int ORDER, int AMODE, int RANGE>
__global__ void __launch_bounds__(256, LBA_FAST_MIN_WAVES) lba_wide_mixed_kernel(const KParams p) { rows_mixed<PM_FLUSH, ORDER, AMODE, RANGE>(p); }

}  // namespace lba
#endif

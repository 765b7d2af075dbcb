// lba_fast_staged.hip -- the smallest forward grids on FP32 carriers under nearest-even: waves of their own that stage.
//
// What bounds such a call (at most one or two workgroups per CU, a lone wave per SIMD) is one wave's issue and the latency of its
// chain, so everything else leaves that wave: lba_fast_kernel's fetches sit behind branches and are waited for where those meet, and
// its decode and stores to LDS run between two parts of the chain.  Four waves run the chains of a 32 x BN tile here (8 rows each,
// BN / 8 columns per lane) and four others fetch, four k-tiles ahead, and decode the k-tile after it; operands lie in groups of
// steps, a 16-byte read each (lba_half_staged_kernel, lba_rows.h, is the same on packed carriers and says why it goes straight through a tile).
// lba_fast_kernel -> parts of 32 steps -> here, us (M = 7; M = 9): 64 x 1000 x 2048 79 -> 41 -> 37 (93 -> 53 -> 50), 300 x 300 x 1500
// 67 -> 30.3 -> 28.0 (77 -> 40 -> 38), 512 x 512 x 512 29.1 -> 23.3 -> 22.1, 64 x 64 x 256 12.9 -> 8.4 -> 8.4.
#include "lba_piece.h"
#include "lba_launch.h"

namespace lba {

template <int N> struct Choice { static constexpr int value = N; };

template <int TN>
struct FastStagedTile {
    static constexpr int BM = 32, BN = 8 * TN, GROUP = 4 / TN;             // steps of B in 16 bytes
    static constexpr int B16 = 16 * BN + 16;                               // 16 steps of B, and a shift of their banks for the lanes that write them
    static constexpr int B_WORDS = HBK / 16 * B16, PITCH = HBK + 4;        // a row of A, and a shift of its banks
    static constexpr int STAGE = B_WORDS + BM * PITCH, STAGES = 4, WORDS = STAGES * STAGE;
};

// The 16 values of a piece, times scale; the two NaN codes read as +-480 (store_tile_cvt).
__device__ __forceinline__ void decode_fp32(const uint4& v, float scale, float (&f)[16]) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t nan_any = 0u;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const v2f lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[d], false), hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[d], true);
        f[4 * d + 0] = lo.x * scale; f[4 * d + 1] = lo.y * scale;
        f[4 * d + 2] = hi.x * scale; f[4 * d + 3] = hi.y * scale;
        nan_any |= ((w[d] & 0x7F7F7F7Fu) + 0x01010101u) & 0x80808080u;     // a byte with low 7 bits all set
    }
    if (nan_any) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const uint32_t code = (w[j >> 2] >> (8 * (j & 3))) & 0xFFu;
            if ((code & 0x7Fu) == 0x7Fu) f[j] = (code & 0x80u) ? -480.0f * scale : 480.0f * scale;
        }
    }
}

// The operands of a lane's chains ahead of the steps (StagedAhead, lba_rows.h): quads of A's values (four steps each) and of B's (GROUP
// steps each), and the products of the step to come.
template <int TN>
struct FastAhead {
    using T = FastStagedTile<TN>;
    static constexpr int G = T::GROUP, STEPS = TN == 2 ? 8 : 4, AQ = STEPS / 4 * 2, BQ = STEPS / G * 2;
    float4 a[AQ], b[BQ];
    float q[TN];
    __device__ __forceinline__ void read_a(const float* base, int i) { a[i % AQ] = *reinterpret_cast<const float4*>(base + 4 * i); }
    __device__ __forceinline__ void read_b(const float* base, int i) { b[i % BQ] = *reinterpret_cast<const float4*>(base + i / (16 / G) * T::B16 + i % (16 / G) * 32); }
    static __device__ __forceinline__ float part(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
    __device__ __forceinline__ float of_a(int k) const { return part(a[k / 4 % AQ], k % 4); }
    __device__ __forceinline__ float of_b(int k, int j) const { return part(b[k / G % BQ], k % G * TN + j); }
    __device__ __forceinline__ void product(int k) {
#pragma unroll
        for (int j = 0; j < TN; ++j) q[j] = of_a(k) * of_b(k, j);   // exact; flushed below Q_prod's R_UF
    }
};

// Steps FROM to FROM + 31 of a tile (staged_steps, lba_rows.h)
template <int PM, int RND, bool CLAMP, int TN, int FROM>
__device__ __forceinline__ void fast_staged_steps(float (&sum)[TN], FastAhead<TN>& o, const float* ab, const float* Bb, const float* an, const float* Bn,
                                                  const FastConst& c) {
    using S = FastAhead<TN>;
#pragma unroll
    for (int k = FROM; k < FROM + 32; ++k) {
        if (k % 4 == 0 || k % S::G == 0) asm volatile("" ::: "memory");   // (reads stay where they are)
        if (k % 4 == 0) {
            const int i = (k + S::STEPS) / 4;
            if (i < HBK / 4) o.read_a(ab, i);
            else             o.read_a(an, i - HBK / 4);
        }
        if (k % S::G == 0) {
            const int i = (k + S::STEPS) / S::G;
            if (i < HBK / S::G) o.read_b(Bb, i);
            else                o.read_b(Bn, i - HBK / S::G);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j)                           // one rounding of the exact sum
            sum[j] = PM == PM_IDENT ? __builtin_fmaf(o.of_a(k), o.of_b(k, j), sum[j]) : __builtin_fmaf(o.q[j], c.kc, sum[j]);
        __builtin_amdgcn_sched_barrier(0);
        if (PM != PM_IDENT) o.product((k + 1) % HBK);
        __builtin_amdgcn_sched_barrier(0);
        if (RND == RND_RNE_BF16) {
#pragma unroll
            for (int j = 0; j < TN; ++j) sum[j] = rne_to_8_bits(sum[j]);
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j) sum[j] = __uint_as_float(rne_bits(__float_as_uint(sum[j]), c.half, c.sh, c.mask));
        }
        if (CLAMP) {
#pragma unroll
            for (int j = 0; j < TN; ++j) sum[j] = med3(sum[j], -c.rof, c.rof);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Row-major E4M3 operands of any alignment, the sequential order; 512 lanes.  TN 4: 32 x 32 tiles, 2: 32 x 16.
template <int TN, int PM, int RND>
__global__ void __launch_bounds__(512, 4) lba_fast_staged_kernel(const KParams p) {
    using T = FastStagedTile<TN>;
    constexpr int AHEAD = kTilesAhead;
    __shared__ __attribute__((aligned(16))) float smem[T::WORDS];
    const int by = TN == 2 ? blockIdx.x / p.mix_gx_tail : blockIdx.y, bx = TN == 2 ? blockIdx.x - by * p.mix_gx_tail : blockIdx.x;
    const int m0 = bx * T::BM, n0 = by * T::BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
    const bool stager = __builtin_amdgcn_readfirstlane(tid >> 8) != 0;
    const int ntiles = (p.K + HBK - 1) / HBK;
    set_flush_f32();

    // A barrier in front of the first tile, which is staged then, and one in the middle of every tile (staged_body, lba_rows.h)
    if (stager) {
        const uint8_t* const pA = p.A + (int64_t)blockIdx.z * p.stride_a;
        const uint8_t* const pB = p.B + (int64_t)blockIdx.z * p.stride_b;
        // waves 0 and 1: 16 rows of A each, four lanes a row; the others: 16 columns of B each (with TN = 2 the last has none)
        const bool isb = wave >= 2;                            // uniform, as all that follows from it
        const int line = (wave & 1) * 16 + (lane >> 2), kq = lane & 3;
        const bool mine = !isb || line < T::BN;
        int rows_a = p.M, rows_b = p.N;
        asm("" : "+s"(rows_a), "+s"(rows_b));                  // (staged_body, lba_rows.h)
        const RowPieces<32> s(isb ? pB : pA, isb ? rows_b : rows_a, p.K, isb ? n0 : m0, mine ? kq * 32 + line : -1);
        const float scale = __builtin_ldexpf(1.0f, isb ? p.exp_b : p.exp_a);
        uint4 r[AHEAD];
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) r[d] = load_piece(s, tile_start(d));   // (a tile beyond K reads codes inside the operands that nothing uses)
        static_assert(AHEAD == T::STAGES, "a tile's stage is its slot of the loads in flight");
        for (int t0 = 0; t0 < ntiles; t0 += AHEAD) {
#pragma unroll
            for (int d = 0; d < AHEAD; ++d) {
                const int t = t0 + d;
                if (t >= ntiles) break;
                float* const st = smem + d * T::STAGE;
                float f[16];
                decode_fp32(s.codes(r[d], t * HBK), scale, f);
                if (!isb) {
                    float4* const row = reinterpret_cast<float4*>(st + T::B_WORDS + line * T::PITCH + kq * 16);
#pragma unroll
                    for (int j = 0; j < 4; ++j) row[j] = make_float4(f[4 * j], f[4 * j + 1], f[4 * j + 2], f[4 * j + 3]);
                } else if (mine) {                             // [k / GROUP][lane of 8][k % GROUP][column]
                    float* const to = st + kq * T::B16 + line / TN * 4 + line % TN;
#pragma unroll
                    for (int j = 0; j < 16; ++j) to[(j / T::GROUP * 8 * T::GROUP + j % T::GROUP) * TN] = f[j];
                }
                r[d] = load_piece(s, tile_start(t + AHEAD));
                __syncthreads();
            }
        }
        __syncthreads();
        return;
    }

    FastConst c;
    c.kc = p.kc; c.rof = p.rof_a; c.mask = p.mask_a; c.half = p.half_a; c.sh = p.sh_a;
    float thresh = p.fast_thresh, thresh4 = p.fast_thresh4;    // fast_body's bounds: below them no sum reaches R_OF in a part of 32 steps, in four,
    float thresh2 = 0.9999f * (2.0f * p.fast_thresh - p.rof_a);   // ... in two: the bound of n parts, R_OF / g^n - n d, is convex in n
    asm volatile("" : "+v"(c.kc), "+v"(c.rof), "+v"(c.mask), "+v"(c.half), "+v"(thresh), "+v"(thresh4), "+v"(thresh2));
    float sum[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) sum[j] = 0.0f;
    const int tx = lane & 7, g = lane >> 3;
    __builtin_amdgcn_s_setprio(3);                             // the chain is what everything waits for
    const float* const Bl = smem + tx * 4;
    const float* const al = smem + T::B_WORDS + (wave * 8 + g) * T::PITCH;
    FastAhead<TN> o;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FastAhead<TN>::STEPS / 4; ++i) o.read_a(al, i);
#pragma unroll
    for (int i = 0; i < FastAhead<TN>::STEPS / T::GROUP; ++i) o.read_b(Bl, i);
    if (PM != PM_IDENT) o.product(0);
    const bool half = ((p.K - 1) & 32) == 0;                   // the last tile's second half lies beyond K (other steps there are products of zeros)
    int t = 0;                                                 // the tile to come
    const auto tiles = [&](auto clamp, int n) {
#pragma unroll 1
        for (n = min(n, ntiles - t); n > 0; --n) {
            const int at = (t & 3) * T::STAGE, then = (++t & 3) * T::STAGE;
            fast_staged_steps<PM, RND, decltype(clamp)::value != 0, TN, 0>(sum, o, al + at, Bl + at, al + then, Bl + then, c);
            __syncthreads();
            if (t == ntiles && half) break;
            fast_staged_steps<PM, RND, decltype(clamp)::value != 0, TN, 32>(sum, o, al + at, Bl + at, al + then, Bl + then, c);
        }
    };
    const auto below = [&](float bound) {
        float mx = 0.0f;
#pragma unroll
        for (int j = 0; j < TN; ++j) mx = __builtin_fmaxf(mx, __builtin_fabsf(sum[j]));
        return __all(mx < bound) != 0;
    };
    while (t < ntiles) {
        if (below(thresh4)) {
            tiles(Choice<0>{}, 2);
        } else if (below(thresh2)) {
            tiles(Choice<0>{}, 1);
        } else if (below(thresh)) {                            // a part at a time
            const int at = (t & 3) * T::STAGE, then = (++t & 3) * T::STAGE;
            fast_staged_steps<PM, RND, false, TN, 0>(sum, o, al + at, Bl + at, al + then, Bl + then, c);
            __syncthreads();
            if (t == ntiles && half) break;
            if (below(thresh)) fast_staged_steps<PM, RND, false, TN, 32>(sum, o, al + at, Bl + at, al + then, Bl + then, c);
            else               fast_staged_steps<PM, RND, true, TN, 32>(sum, o, al + at, Bl + at, al + then, Bl + then, c);
        } else {
            tiles(Choice<1>{}, 2);
        }
    }
    // C = S * 2^out_exp, zero written as +0
    const int m = m0 + wave * 8 + g, n = n0 + tx * TN;
    if (m >= p.M) return;
    float* const dst = p.C + (int64_t)blockIdx.z * p.stride_c + (int64_t)m * p.N + n;
    float v[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) v[j] = sum[j] == 0.0f ? 0.0f : __builtin_ldexpf(sum[j], p.out_exp);
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

template <int PM, int RND>
static hipError_t launch_one(const Plan& pl, hipStream_t st) {
    const dim3 grid(pl.grid_x, pl.grid_y, pl.kp.batch), block(512);
    if (pl.mix_tail > 0) hipLaunchKernelGGL((lba_fast_staged_kernel<2, PM, RND>), grid, block, 0, st, pl.kp);
    else                 hipLaunchKernelGGL((lba_fast_staged_kernel<4, PM, RND>), grid, block, 0, st, pl.kp);
    return hipGetLastError();
}

hipError_t launch_fast_staged(const Plan& pl, hipStream_t st) {
    if (pl.events || pl.round != LBA_ROUND_RNE || pl.rne_odd || pl.amode || pl.kp.conv || pl.kp.h_on || pl.order != LBA_ORDER_SEQ || pl.bk != 32) return hipErrorInvalidValue;
    if (pl.mix_tail > 0 ? !pl.kp.mix_tail16 || pl.kp.mix_main + pl.kp.mix_half != 0 : pl.tm != 2 || pl.tn != 2) return hipErrorInvalidValue;
    if (pl.prod_mode == PM_IDENT) return pl.kp.sh_a == 16 ? launch_one<PM_IDENT, RND_RNE_BF16>(pl, st) : launch_one<PM_IDENT, LBA_ROUND_RNE>(pl, st);
    if (pl.prod_mode == PM_FLUSH) return pl.kp.sh_a == 16 ? launch_one<PM_FLUSH, RND_RNE_BF16>(pl, st) : launch_one<PM_FLUSH, LBA_ROUND_RNE>(pl, st);
    return hipErrorInvalidValue;
}

}  // namespace lba

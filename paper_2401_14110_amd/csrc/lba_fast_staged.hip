// lba_fast_staged.hip -- the smallest forward grids on FP32 carriers under nearest-even: waves of their own that stage.
//
// What bounds such a call (at most one or two workgroups per CU, a lone wave per SIMD) is one wave's issue and the latency of its
// chain, so everything else leaves that wave: lba_fast_kernel's fetches sit behind branches and are waited for where those meet, and
// its decode and stores to LDS run between two parts of the chain.  Four waves run the chains of a 32 x BN tile here (8 rows each,
// BN / 8 columns per lane) and four others fetch, four k-tiles ahead, and decode the k-tile after it; operands lie in groups of
// steps, a 16-byte read each (lba_half_staged_kernel, lba_rows.h, is the same on packed carriers).
// lba_fast_kernel -> here, us (M = 7; M = 9): 64 x 64 x 256 12.9 -> 8.6 (14.7 -> 10.2), 64 x 1000 x 2048 79 -> 48 (93 -> 61), 300 x 300 x 1500
// 67 -> 37 (77 -> 46), 512 x 512 x 512 29.1 -> 23.5, 128 x 4096 x 1024 (512 workgroups) 75 -> 65, 64 x 64 x 64 7.7 -> 7.6.
#include "lba_piece.h"
#include "lba_launch.h"

namespace lba {

template <int TN>
struct FastStagedTile {
    static constexpr int BM = 32, BN = 8 * TN, GROUP = 4 / TN;             // steps of B in 16 bytes
    static constexpr int B_WORDS = HBK * BN, PITCH = HBK + 4;              // a row of A, and a shift of its banks
    static constexpr int STAGE = B_WORDS + BM * PITCH, WORDS = 2 * STAGE;
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

// 32 steps of the lane's chains; operands are read eight steps ahead, products taken before the sum ahead of them is rounded.
template <int PM, int RND, bool CLAMP, int TN>
__device__ __forceinline__ void fast_staged_steps(float (&sum)[TN], const float* arow, const float* Bs, const FastConst& c) {
    constexpr int G = FastStagedTile<TN>::GROUP, GROUPS = 32 / G, AHEAD = 8 / G;
    float4 a[8], b[GROUPS];
    float q[2][TN];
    auto part = [](const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; };
    auto product = [&](int k) {
#pragma unroll
        for (int j = 0; j < TN; ++j) q[k & 1][j] = part(a[k / 4], k % 4) * part(b[k / G], k % G * TN + j);   // exact; flushed below Q_prod's R_UF
    };
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const float4*>(arow + 4 * i);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) b[i] = *reinterpret_cast<const float4*>(Bs + i * 32);
    if (PM != PM_IDENT) product(0);
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        if (k % 4 == 0 && k / 4 + 2 < 8) a[k / 4 + 2] = *reinterpret_cast<const float4*>(arow + k + 8);
        if (k % G == 0 && k / G + AHEAD < GROUPS) b[k / G + AHEAD] = *reinterpret_cast<const float4*>(Bs + (k / G + AHEAD) * 32);
#pragma unroll
        for (int j = 0; j < TN; ++j)                           // one rounding of the exact sum
            sum[j] = PM == PM_IDENT ? __builtin_fmaf(part(a[k / 4], k % 4), part(b[k / G], k % G * TN + j), sum[j]) : __builtin_fmaf(q[k & 1][j], c.kc, sum[j]);
        __builtin_amdgcn_sched_barrier(0);
        if (PM != PM_IDENT && k < 31) product(k + 1);
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

    // One barrier a tile: behind it the tile is staged and the stage before it no longer read.
    if (stager) {
        const uint8_t* const pA = p.A + (int64_t)blockIdx.z * p.stride_a;
        const uint8_t* const pB = p.B + (int64_t)blockIdx.z * p.stride_b;
        // lanes 0 .. 31: pieces of the wave's 8 rows of A; 32 and up: pieces of B, 16 steps a wave
        const bool isb = lane >= 32;
        const int ca = isb ? -1 : (lane & 3) * T::BM + wave * 8 + (lane >> 2), cb = isb && lane - 32 < T::BN ? wave * T::BN + lane - 32 : -1;
        RowPieces<T::BM> s(pA, p.M, p.K, m0, ca);
        const RowPieces<T::BN> sb(pB, p.N, p.K, n0, cb);
        if (isb) { s.row = sb.row; s.kq = sb.kq; s.room = sb.room; s.end = sb.end; s.ok = sb.ok; }
        const float scale = __builtin_ldexpf(1.0f, isb ? p.exp_b : p.exp_a);
        uint4 r[AHEAD];
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) r[d] = load_piece(s, tile_start(d));   // (a tile beyond K reads codes inside the operands that nothing uses)
        for (int t0 = 0; t0 < ntiles; t0 += AHEAD) {
#pragma unroll
            for (int d = 0; d < AHEAD; ++d) {
                const int t = t0 + d;
                if (t >= ntiles) break;
                float* const st = smem + (t & 1) * T::STAGE;
                float f[16];
                decode_fp32(s.codes(r[d], t * HBK), scale, f);
                if (!isb) {
                    float4* const row = reinterpret_cast<float4*>(st + T::B_WORDS + (wave * 8 + (lane >> 2)) * T::PITCH + (lane & 3) * 16);
#pragma unroll
                    for (int j = 0; j < 4; ++j) row[j] = make_float4(f[4 * j], f[4 * j + 1], f[4 * j + 2], f[4 * j + 3]);
                } else if (cb >= 0) {                          // [k / GROUP][lane of 8][k % GROUP][column]
                    const int col = lane - 32;
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const int k = wave * 16 + j;
                        st[((k / T::GROUP * 8 + col / TN) * T::GROUP + k % T::GROUP) * TN + col % TN] = f[j];
                    }
                }
                r[d] = load_piece(s, tile_start(t + AHEAD));
                __syncthreads();
            }
        }
        return;
    }

    FastConst c;
    c.kc = p.kc; c.rof = p.rof_a; c.mask = p.mask_a; c.half = p.half_a; c.sh = p.sh_a;
    float thresh = p.fast_thresh, thresh4 = p.fast_thresh4;
    asm volatile("" : "+v"(c.kc), "+v"(c.rof), "+v"(c.mask), "+v"(c.half), "+v"(thresh), "+v"(thresh4));
    float sum[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) sum[j] = 0.0f;
    const int tx = lane & 7, g = lane >> 3;
    int safe_tiles = 0;
    __builtin_amdgcn_s_setprio(3);                             // the chain is what everything waits for
    for (int t = 0; t < ntiles; ++t) {
        __syncthreads();
        const float* const Bs = smem + (t & 1) * T::STAGE + tx * 4;
        const float* const arow = smem + (t & 1) * T::STAGE + T::B_WORDS + (wave * 8 + g) * T::PITCH;
        const int parts = p.K - t * HBK > 32 ? 2 : 1;
        for (int part = 0; part < parts; ++part) {
            if (safe_tiles == 0) {                             // fast_body's bound: no sum reaches R_OF in that many tiles of 32 steps
                float mx = 0.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j) mx = __builtin_fmaxf(mx, __builtin_fabsf(sum[j]));
                safe_tiles = __all(mx < thresh4) ? 4 : (__all(mx < thresh) ? 1 : 0);
            }
            const float* const Bp = Bs + part * (T::B_WORDS / 2);
            if (safe_tiles > 0) {
                --safe_tiles;
                fast_staged_steps<PM, RND, false, TN>(sum, arow + part * 32, Bp, c);
            } else {
                fast_staged_steps<PM, RND, true, TN>(sum, arow + part * 32, Bp, c);
            }
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

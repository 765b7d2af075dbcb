// lba_piece.h -- how a lane of the packed FP16 tiles fetches its 16-code pieces: a load that nothing depends on until the
// piece is staged, then the correction of what it read.  The load is unconditional, from an address inside the operand, so it
// sits in straight-line code and stays in flight over the k-tiles between (loads behind branches, merged with a zero, were
// waited for where the branches met).
#ifndef LBA_PIECE_H_
#define LBA_PIECE_H_

#include "lba_device.h"

namespace lba {

struct Bytes16 { uint64_t lo, hi; };

__device__ __forceinline__ Bytes16 as_bytes(const uint4& v) {
    return {(uint64_t)v.x | ((uint64_t)v.y << 32), (uint64_t)v.z | ((uint64_t)v.w << 32)};
}
__device__ __forceinline__ uint4 as_uint4(const Bytes16& b) {
    return make_uint4((uint32_t)b.lo, (uint32_t)(b.lo >> 32), (uint32_t)b.hi, (uint32_t)(b.hi >> 32));
}
// byte j of the result is byte j + s of b, zero outside; -16 <= s <= 16
__device__ __forceinline__ Bytes16 shift_bytes(Bytes16 b, int s) {
    const int n = s < 0 ? -s : s, bits = (n & 7) * 8;
    if (s >= 0) {
        if (n & 8) { b.lo = b.hi; b.hi = 0; }
        if (bits) { b.lo = (b.lo >> bits) | (b.hi << (64 - bits)); b.hi >>= bits; }
    } else {
        if (n & 8) { b.hi = b.lo; b.lo = 0; }
        if (bits) { b.hi = (b.hi << bits) | (b.lo >> (64 - bits)); b.lo <<= bits; }
    }
    if (n & 16) b = {0, 0};
    return b;
}
// the low n bytes of a word, n clamped to 0 .. 8
__device__ __forceinline__ uint64_t low_bytes(int n) { return n >= 8 ? ~0ull : (n <= 0 ? 0ull : ((1ull << (8 * n)) - 1ull)); }
// bytes [from, to) of b, zero elsewhere
__device__ __forceinline__ Bytes16 keep_bytes(const Bytes16& b, int from, int to) {
    return {b.lo & low_bytes(to) & ~low_bytes(from), b.hi & low_bytes(to - 8) & ~low_bytes(from - 8)};
}

// A piece of a matrix whose rows are 16-byte aligned (K % 16 == 0), zero outside the matrix.
template <int ROWS>
__device__ __forceinline__ uint4 fetch_aligned(const uint8_t* __restrict__ G, int rows, int K, int r0, int k0, int c) {
    const int r = r0 + c % ROWS, k = k0 + c / ROWS * 16;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (c >= 0 && c < Stage<ROWS, 64>::kChunks && r < rows && k < K) v = *reinterpret_cast<const uint4*>(G + (int64_t)r * K + k);
    return v;
}

// A piece of im2col rows whose 16 codes are channels of one tap (fetch_tile_conv_lane's aligned case).
__device__ __forceinline__ uint4 fetch_taps(const ConvLane& L, const KParams& p, int k0) {
    const int k = k0 + L.kq16;
    const int tap = (int)div_magic((uint32_t)k, p.cv_magic_c), ch = k - tap * p.cv_c;
    const int kh = (int)div_magic((uint32_t)tap, p.cv_magic_kw), kw = tap - kh * p.cv_kw;
    const int ih = L.ih0 + kh, iw = L.iw0 + kw;
    const bool in = L.ok && k < p.K && (unsigned)ih < (unsigned)p.cv_h && (unsigned)iw < (unsigned)p.cv_w;
    const int64_t off = in ? ((int64_t)ih * p.cv_w + iw) * p.cv_c + ch : 0;       // (an image holds 16 bytes or more)
    const uint4 v = *reinterpret_cast<const uint4*>(L.img + off);
    return make_uint4(in ? v.x : 0u, in ? v.y : 0u, in ? v.z : 0u, in ? v.w : 0u);
}

// A row-major matrix [rows][K] at G; the lane's piece c of a tile of ROWS rows from r0: row c % ROWS, codes 16 (c / ROWS) ...
template <int ROWS>
struct RowPieces {
    const uint8_t* row;        // the lane's row (a row of the matrix in any case)
    const uint8_t* last;       // the last address from which 16 bytes lie inside the matrix (which holds at least 16)
    int K, kq;
    bool ok, whole;            // the row exists; K % 16 == 0 (uniform): every piece is inside its row or beyond it

    __device__ __forceinline__ RowPieces(const uint8_t* G, int rows, int K_, int r0, int c) {
        const int r = r0 + c % ROWS;
        ok = c >= 0 && c < Stage<ROWS, 64>::kChunks && r < rows;
        K = K_;
        kq = c >= 0 ? c / ROWS * 16 : 0;
        row = G + (int64_t)(ok ? r : 0) * K;
        last = G + ((int64_t)rows * K - 16);
        whole = (K & 15) == 0;
    }
    __device__ __forceinline__ uint4 load(int k0) const {
        const uint8_t* p = row + min(k0 + kq, K);
        const u32x4_bytes x = *reinterpret_cast<const u32x4_bytes*>(p < last ? p : last);
        return make_uint4(x.x, x.y, x.z, x.w);
    }
    // the codes of the tile at k0 in what load(k0) returned: zero beyond the row and outside the matrix
    __device__ __forceinline__ uint4 codes(uint4 v, int k0) const {
        const int n = ok ? K - (k0 + kq) : 0;                  // codes left in the row
        if (whole) return make_uint4(n > 0 ? v.x : 0u, n > 0 ? v.y : 0u, n > 0 ? v.z : 0u, n > 0 ? v.w : 0u);
        if (n < 16) {
            const int back = (int)(row + (k0 + kq) - last);    // > 0: the load started that many bytes early
            Bytes16 b = as_bytes(v);
            if (n > 0 && back > 0) b = shift_bytes(b, back);
            v = as_uint4(keep_bytes(b, 0, n));
        }
        return v;
    }
};

// im2col rows of an NHWC tensor (see fetch_tile_conv_lane).  C % 16 == 0 and X aligned: a piece is 16 channels of one tap.
// Otherwise the codes of one filter row, KW * C of them, are contiguous in memory, and a piece spans at most two filter rows
// when KW * C >= 16: two unaligned loads (the first convolution of a ResNet, C = 3: sixteen byte loads before).
struct ConvPieces {
    const uint8_t* X;
    const uint8_t* img;        // X + n * H * W * C
    const uint8_t* last;       // the last address from which 16 bytes lie inside the tensor (which holds at least 16)
    int ih0, iw0, kq;
    bool ok, spans;

    template <int ROWS>
    static __device__ __forceinline__ ConvPieces make(const uint8_t* X, const KParams& p, int r0, int c) {
        ConvPieces s;
        const int r = r0 + c % ROWS;
        s.ok = c >= 0 && c < Stage<ROWS, 64>::kChunks && r < p.M;
        const int rr = s.ok ? r : 0;
        const int ow = rr % p.cv_ow, t = rr / p.cv_ow;
        const int oh = t % p.cv_oh, n = t / p.cv_oh;
        const int64_t image = (int64_t)p.cv_h * p.cv_w * p.cv_c, total = image * (p.M / (p.cv_oh * p.cv_ow));
        s.X = X;
        s.img = X + n * image;
        s.last = X + (total - 16);
        s.ih0 = oh * p.cv_stride - p.cv_pad;
        s.iw0 = ow * p.cv_stride - p.cv_pad;
        s.kq = c >= 0 ? c / ROWS * 16 : 0;
        s.spans = p.cv_kw * p.cv_c >= 16;                      // uniform
        return s;
    }
    struct At { int kh, r; };                                  // filter row of code k, its position among that row's KW * C codes
    __device__ __forceinline__ At at(const KParams& p, int k) const {
        const int tap = (int)div_magic((uint32_t)k, p.cv_magic_c);
        const int kh = (int)div_magic((uint32_t)tap, p.cv_magic_kw);
        return {kh, k - kh * p.cv_kw * p.cv_c};
    }
    // bytes of the filter row's run that lie inside the image: [lo, hi)
    __device__ __forceinline__ bool inside(const KParams& p, int kh, int& lo, int& hi) const {
        lo = iw0 < 0 ? -iw0 * p.cv_c : 0;
        hi = min(p.cv_kw, p.cv_w - iw0) * p.cv_c;
        return ok && (unsigned)(ih0 + kh) < (unsigned)p.cv_h;
    }
    __device__ __forceinline__ const uint8_t* address(const KParams& p, int kh, int r) const {
        return img + ((int64_t)(ih0 + kh) * p.cv_w + iw0) * p.cv_c + r;
    }
    __device__ __forceinline__ const uint8_t* clamped(const uint8_t* a) const { return a < X ? X : (a > last ? last : a); }

    __device__ __forceinline__ uint4 load_at(const uint8_t* a) const {
        const u32x4_bytes x = *reinterpret_cast<const u32x4_bytes*>(clamped(a));
        return make_uint4(x.x, x.y, x.z, x.w);
    }
    __device__ __forceinline__ void load(const KParams& p, int k0, uint4& u, uint4& v) const {
        const At a = at(p, k0 + kq);
        u = load_at(address(p, a.kh, a.r));
        if (!p.cv_vec) v = load_at(address(p, a.kh + 1, 0));   // uniform
    }
    __device__ __forceinline__ uint4 codes(const KParams& p, const uint4& u, const uint4& v, int k0) const {
        if (p.cv_vec) {                                        // uniform: one tap
            const int k = k0 + kq;
            const At a = at(p, k);
            const int iw = iw0 + (int)div_magic((uint32_t)a.r, p.cv_magic_c);
            const bool in = ok && k < p.K && (unsigned)(ih0 + a.kh) < (unsigned)p.cv_h && (unsigned)iw < (unsigned)p.cv_w;
            return in ? u : make_uint4(0u, 0u, 0u, 0u);
        }
        if (!spans) {                                          // uniform: a few channels under a narrow filter, byte by byte
            Bytes16 b = {0, 0};
#pragma unroll 1
            for (int j = 0; j < 16; ++j) {
                const int k = k0 + kq + j;
                const At e = at(p, k);
                int lo, hi;
                if (k < p.K && inside(p, e.kh, lo, hi) && e.r >= lo && e.r < hi)
                    (j < 8 ? b.lo : b.hi) |= (uint64_t)*address(p, e.kh, e.r) << (8 * (j & 7));
            }
            return as_uint4(b);
        }
        const int k = k0 + kq, n = min(16, p.K - k);           // codes of the piece below K
        const At a = at(p, k);
        const int n1 = min(n, p.cv_kw * p.cv_c - a.r);         // of them in the first filter row
        Bytes16 x = {0, 0}, y = {0, 0};
        int lo, hi;
        if (n > 0 && inside(p, a.kh, lo, hi)) {
            const uint8_t* q = address(p, a.kh, a.r);
            x = keep_bytes(shift_bytes(as_bytes(u), (int)(q - clamped(q))), lo - a.r, min(n1, hi - a.r));
        }
        if (n > n1 && inside(p, a.kh + 1, lo, hi)) {
            const uint8_t* q = address(p, a.kh + 1, 0);
            y = shift_bytes(keep_bytes(shift_bytes(as_bytes(v), (int)(q - clamped(q))), lo, min(n - n1, hi)), -n1);
        }
        return as_uint4({x.lo | y.lo, x.hi | y.hi});
    }
};

}  // namespace lba
#endif

// lba_piece_index.h -- which 16 bytes of an operand a lane of the packed FP16 tiles loads for a 16-code piece, and which codes
// of the piece are in them (lba_piece.h does the loads).  Plain C++: tests/sanitize_pieces.cpp runs this arithmetic on the host
// at the ends of the shape limits, where 32-bit products and differences would wrap.
#ifndef LBA_PIECE_INDEX_H_
#define LBA_PIECE_INDEX_H_

#include <stdint.h>

#include "lba_internal.h"

#if defined(__HIP__)
#define LBA_HOST_DEVICE __attribute__((host, device, always_inline)) inline
#else
#define LBA_HOST_DEVICE inline
#endif

namespace lba {

enum { HBK = 64 };                                             // steps of a k-tile of the packed tiles

LBA_HOST_DEVICE uint32_t div_magic(uint32_t x, uint64_t magic) { return (uint32_t)(((uint64_t)x * magic) >> 40); }

struct Bytes16 { uint64_t lo, hi; };

template <class V>
LBA_HOST_DEVICE Bytes16 as_bytes(const V& v) {
    return {(uint64_t)v.x | ((uint64_t)v.y << 32), (uint64_t)v.z | ((uint64_t)v.w << 32)};
}
template <class V>
LBA_HOST_DEVICE V as_words(const Bytes16& b) {
    V v;
    v.x = (uint32_t)b.lo; v.y = (uint32_t)(b.lo >> 32); v.z = (uint32_t)b.hi; v.w = (uint32_t)(b.hi >> 32);
    return v;
}
// byte j of the result is byte j + s of b, zero outside; -16 <= s <= 16
LBA_HOST_DEVICE Bytes16 shift_bytes(Bytes16 b, int s) {
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
LBA_HOST_DEVICE uint64_t low_bytes(int n) { return n >= 8 ? ~0ull : (n <= 0 ? 0ull : ((1ull << (8 * n)) - 1ull)); }
// bytes [from, to) of b, zero elsewhere
LBA_HOST_DEVICE Bytes16 keep_bytes(const Bytes16& b, int from, int to) {
    return {b.lo & low_bytes(to) & ~low_bytes(from), b.hi & low_bytes(to - 8) & ~low_bytes(from - 8)};
}

// First k of tile t, also of the up to four tiles beyond the last one that are fetched ahead and never used: every k of those
// stays below 2^31 where K is at most kPieceMaxK, and the planner keeps longer chains on the FP32 tile, which fetches no tile
// beyond the last one.  (Clamping t, or unsigned arithmetic, in the small lane blocks' loop instead: 64 x 1000 x 2048 44.9 ->
// 45.4 and 45.8 us.)
enum { kTilesAhead = 4 };
constexpr int64_t kPieceMaxK = ((int64_t)1 << 31) - (kTilesAhead + 1) * HBK;
LBA_HOST_DEVICE int tile_start(int t) { return t * HBK; }

// A row-major matrix [rows][K] at G; the lane's piece c of a tile of ROWS rows from r0: row c % ROWS, codes 16 (c / ROWS) ...
template <int ROWS>
struct RowPieces {
    const uint8_t* row;        // the lane's row (a row of the matrix in any case)
    int K, kq;
    int room;                  // the last k from which 16 bytes lie inside the matrix (which holds at least 16): -15 or more, and
                               // taken as 2^31 - 1 where it is larger
    int end;                   // of K and room the smaller
    bool ok, whole;            // the row exists; K % 16 == 0 (uniform): every piece is inside its row or beyond it

    LBA_HOST_DEVICE RowPieces(const uint8_t* G, int rows, int K_, int r0, int c) {
        const int r = r0 + c % ROWS;
        ok = c >= 0 && c < ROWS * HBK / 16 && r < rows;
        K = K_;
        kq = c >= 0 ? c / ROWS * 16 : 0;
        row = G + (int64_t)(ok ? r : 0) * K;
        const int64_t left = (int64_t)(rows - (ok ? r : 0)) * K - 16;
        room = left < 0x7FFFFFFF ? (int)left : 0x7FFFFFFF;
        end = K < room ? K : room;
        whole = (K & 15) == 0;
    }
    // where the 16 bytes of the tile at k0 are loaded from
    LBA_HOST_DEVICE const uint8_t* address(int k0) const {
        const int k = k0 + kq;
        return row + (k < end ? k : end);
    }
    // the codes of the tile at k0 in what address(k0) holds: zero beyond the row and outside the matrix
    template <class V>
    LBA_HOST_DEVICE V codes(V v, int k0) const {
        const int n = ok ? K - (k0 + kq) : 0;                  // codes left in the row
        if (whole) {
            v.x = n > 0 ? v.x : 0u; v.y = n > 0 ? v.y : 0u; v.z = n > 0 ? v.z : 0u; v.w = n > 0 ? v.w : 0u;
            return v;
        }
        if (n < 16) {
            const int back = k0 + kq - room;                   // > 0: the load started that many bytes early (15 at most)
            Bytes16 b = as_bytes(v);
            if (n > 0 && back > 0) b = shift_bytes(b, back);
            v = as_words<V>(keep_bytes(b, 0, n));
        }
        return v;
    }
};

// im2col rows of an NHWC tensor (see fetch_tile_conv_lane).  C % 16 == 0 and X aligned: a piece is 16 channels of one tap.
// Otherwise the codes of one filter row, KW * C of them, are contiguous in memory, and a piece spans at most two filter rows
// when KW * C >= 16: two unaligned loads (the first convolution of a ResNet, C = 3: sixteen byte loads before).
struct ConvPieces {
    const uint8_t* X;
    int64_t img;               // n * H * W * C
    int64_t last;              // the last offset from which 16 bytes lie inside the tensor (which holds at least 16)
    int ih0, iw0, kq;
    int lo, hi;                // of a filter row's KW * C codes, those inside the image's columns: [lo, hi)
    bool ok, spans;

    // Columns are compared as columns: the padding is not limited, so iw0 * C (or W - iw0) can pass 2^31.  ih0 and iw0 are taken
    // modulo 2^32 (unsigned arithmetic): one that wraps lies 2^31 or more beyond the image, wraps to a negative number and stays
    // outside.
    template <int ROWS>
    static LBA_HOST_DEVICE ConvPieces make(const uint8_t* X, const KParams& p, int r0, int c) {
        ConvPieces s;
        const int r = r0 + c % ROWS;
        s.ok = c >= 0 && c < ROWS * HBK / 16 && r < p.M;
        const int rr = s.ok ? r : 0;
        const int ow = rr % p.cv_ow, t = rr / p.cv_ow;
        const int oh = t % p.cv_oh, n = t / p.cv_oh;
        const int64_t image = (int64_t)p.cv_h * p.cv_w * p.cv_c, total = image * (p.M / (p.cv_oh * p.cv_ow));
        s.X = X;
        s.img = n * image;
        s.last = total - 16;
        s.ih0 = (int)((uint32_t)oh * (uint32_t)p.cv_stride - (uint32_t)p.cv_pad);
        s.iw0 = (int)((uint32_t)ow * (uint32_t)p.cv_stride - (uint32_t)p.cv_pad);
        s.kq = c >= 0 ? c / ROWS * 16 : 0;
        const int left = s.iw0 >= 0 ? 0 : (s.iw0 > -p.cv_kw ? -s.iw0 : p.cv_kw);              // taps left of the image
        const int right = s.iw0 <= p.cv_w - p.cv_kw ? p.cv_kw : (s.iw0 < p.cv_w ? p.cv_w - s.iw0 : 0);   // taps not right of it
        s.lo = left * p.cv_c;
        s.hi = right * p.cv_c;
        s.spans = p.cv_kw * p.cv_c >= 16;                      // uniform
        return s;
    }
    struct At { int kh, r; };                                  // filter row of code k, its position among that row's KW * C codes
    LBA_HOST_DEVICE At at(const KParams& p, int k) const {
        const int tap = (int)div_magic((uint32_t)k, p.cv_magic_c);
        const int kh = (int)div_magic((uint32_t)tap, p.cv_magic_kw);
        return {kh, k - kh * p.cv_kw * p.cv_c};
    }
    LBA_HOST_DEVICE bool inside(const KParams& p, int kh) const { return ok && (uint32_t)ih0 + (uint32_t)kh < (uint32_t)p.cv_h; }
    // offset of code r of filter row kh (meaningful, and free of wraps, for a row inside the image)
    LBA_HOST_DEVICE int64_t offset(const KParams& p, int kh, int r) const {
        const uint64_t ih = (uint64_t)(int64_t)(int)((uint32_t)ih0 + (uint32_t)kh);
        return img + (int64_t)((ih * (uint64_t)p.cv_w + (uint64_t)(int64_t)iw0) * (uint64_t)p.cv_c + (uint64_t)r);
    }
    LBA_HOST_DEVICE int64_t clamped(int64_t a) const { return a < 0 ? 0 : (a > last ? last : a); }
    // how many bytes before a its clamped load started (< 0: after it): at most 15 where any of the piece's codes are inside the
    // image, and anything from -16 to 15 (the difference's low five bits) where none are and nothing is kept
    LBA_HOST_DEVICE int early(int64_t a) const { return (int32_t)((uint32_t)(uint64_t)(a - clamped(a)) << 27) >> 27; }
    // where the two loads of the tile at k0 start: at its first code, and at the next filter row
    LBA_HOST_DEVICE const uint8_t* first(const KParams& p, int k0) const {
        const At a = at(p, k0 + kq);
        return X + clamped(offset(p, a.kh, a.r));
    }
    LBA_HOST_DEVICE const uint8_t* second(const KParams& p, int k0) const { return X + clamped(offset(p, at(p, k0 + kq).kh + 1, 0)); }

    // the same where p.cv_vec: one tap
    template <class V>
    LBA_HOST_DEVICE V tap_codes(const KParams& p, const V& u, int k0) const {
        const int k = k0 + kq;
        const At a = at(p, k);
        const bool in = k < p.K && inside(p, a.kh) && a.r >= lo && a.r < hi;
        return in ? u : as_words<V>({0, 0});
    }
    // the codes of the tile at k0 in what first(k0) and second(k0) hold (v is not read where p.cv_vec)
    template <class V>
    LBA_HOST_DEVICE V codes(const KParams& p, const V& u, const V& v, int k0) const {
        if (p.cv_vec) return tap_codes(p, u, k0);              // uniform
        if (!spans) {                                          // uniform: a few channels under a narrow filter, byte by byte
            Bytes16 b = {0, 0};
#pragma unroll 1
            for (int j = 0; j < 16; ++j) {
                const int k = k0 + kq + j;
                const At e = at(p, k);
                if (k < p.K && inside(p, e.kh) && e.r >= lo && e.r < hi)
                    (j < 8 ? b.lo : b.hi) |= (uint64_t)X[offset(p, e.kh, e.r)] << (8 * (j & 7));
            }
            return as_words<V>(b);
        }
        return row_codes(p, u, v, k0);
    }
    // the same for filter rows that a piece may span, two at most (spans)
    template <class V>
    LBA_HOST_DEVICE V row_codes(const KParams& p, const V& u, const V& v, int k0) const {
        const int k = k0 + kq, n = p.K - k < 16 ? p.K - k : 16;   // codes of the piece below K
        const At a = at(p, k);
        const int left = p.cv_kw * p.cv_c - a.r, n1 = n < left ? n : left;   // of them in the first filter row
        Bytes16 x = {0, 0}, y = {0, 0};
        if (n > 0 && inside(p, a.kh)) {
            x = keep_bytes(shift_bytes(as_bytes(u), early(offset(p, a.kh, a.r))), lo - a.r, n1 < hi - a.r ? n1 : hi - a.r);
        }
        if (n > n1 && inside(p, a.kh + 1)) {
            y = shift_bytes(keep_bytes(shift_bytes(as_bytes(v), early(offset(p, a.kh + 1, 0))), lo, n - n1 < hi ? n - n1 : hi), -n1);
        }
        return as_words<V>({x.lo | y.lo, x.hi | y.hi});
    }
};

}  // namespace lba
#endif

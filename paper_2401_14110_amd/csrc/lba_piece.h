// lba_piece.h -- how a lane of the packed FP16 tiles fetches its 16-code pieces: a load that nothing depends on until the
// piece is staged, then the correction of what it read (lba_piece_index.h has the addresses and the corrections).  The load is
// unconditional, from an address inside the operand, so it sits in straight-line code and stays in flight over the k-tiles
// between (loads behind branches, merged with a zero, were waited for where the branches met).
#ifndef LBA_PIECE_H_
#define LBA_PIECE_H_

#include "lba_device.h"
#include "lba_piece_index.h"

namespace lba {

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

__device__ __forceinline__ uint4 load_16(const uint8_t* a) {   // any alignment
    const u32x4_bytes x = *reinterpret_cast<const u32x4_bytes*>(a);
    return make_uint4(x.x, x.y, x.z, x.w);
}

template <int ROWS>
__device__ __forceinline__ uint4 load_piece(const RowPieces<ROWS>& s, int k0) { return load_16(s.address(k0)); }

__device__ __forceinline__ void load_piece(const ConvPieces& s, const KParams& p, int k0, uint4& u, uint4& v) {
    u = load_16(s.first(p, k0));
    if (!p.cv_vec) v = load_16(s.second(p, k0));               // uniform
}

}  // namespace lba
#endif

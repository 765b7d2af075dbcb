"""The plans that the entry points launch (tests/launch_recorder.cpp), on the host: grids that fit the kernel's tiles, and the plan of the planes asked for."""
import ctypes
import os
import subprocess

import pytest

from paper_2401_14110_amd.binding import lba_conv2d_desc, lba_infmt, lba_qfmt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FIELDS = ("grid_x", "grid_y", "tm", "tn", "mix_main", "mix_half", "mix_tail", "mix_tail16", "packed", "staged", "alone", "of_only", "kpar")


class Launched(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in FIELDS]


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("launches") / "launch_recorder.so")
    csrc = os.path.join(ROOT, "paper_2401_14110_amd", "csrc")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O1", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "lba_kernels.hip"), os.path.join(csrc, "lba_plan.cpp"),
                    os.path.join(ROOT, "tests", "launch_recorder.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    vp, i64, i32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32
    lib.take_launched.restype = ctypes.c_char_p
    lib.lba_conv2d.argtypes = [vp, vp, vp, lba_conv2d_desc, i64, lba_qfmt, lba_qfmt, i32, vp]
    lib.lba_conv2d_bwd.argtypes = [vp, vp, vp, vp, vp, lba_conv2d_desc, i64, lba_qfmt, lba_qfmt, i32, vp]
    lib.lba_gemm.argtypes = [vp, vp, vp, i64, i64, i64, lba_qfmt, lba_qfmt, i32, vp]
    lib.lba_gemm_bwd.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, lba_qfmt, lba_qfmt, i32, vp]
    lib.lba_gemm_bwd_chunked.argtypes = [vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, lba_qfmt, lba_qfmt, vp]
    lib.lba_gemm_batched.argtypes = [vp, vp, vp, i64, i64, i64, i64, i64, i64, i64, lba_qfmt, lba_qfmt, i32, vp]
    lib.lba_gemm_bwd_in.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, lba_infmt, lba_infmt, lba_qfmt, lba_qfmt, i32, vp]
    return lib


def taken(lib):
    out = Launched()
    name = lib.take_launched(ctypes.byref(out)).decode()
    return name, {n: getattr(out, n) for n in FIELDS}


BUF = 1 << 20        # (never read: an address on a 16-byte boundary)
PACKED, TRUNC = ((5, 7, 12, 0), (4, 7, 9, 0)), ((5, 4, 12, 0), (4, 7, 9, 0))


def conv(lib, n, h, w, c, cout, k, formats, planes, order=0):
    d = lba_conv2d_desc(n, h, w, c, k, k, 1, k // 2)
    qp, qa = (lba_qfmt(*f) for f in formats)
    if planes is None:
        rc = lib.lba_conv2d(BUF, BUF, BUF, d, cout, qp, qa, order, None)
    else:
        rc = lib.lba_conv2d_bwd(BUF, BUF, BUF, BUF if "o" in planes else None, BUF if "u" in planes else None, d, cout, qp, qa, order, None)
    assert rc == 0
    o = h + 2 * (k // 2) - k + 1, w + 2 * (k // 2) - k + 1
    return (n * o[0] * o[1], cout) + taken(lib)


def fits(M, N, p):
    """A plain grid of the plan's tiles, or the mixed grid's regions."""
    up = lambda a, b: -(-a // b)  # noqa: E731
    if p["mix_tail"] == 0:
        return (p["grid_x"], p["grid_y"]) == (up(M, 16 * p["tm"]), up(N, 16 * p["tn"]))
    return p["grid_x"] == p["mix_main"] + p["mix_tail"] and p["grid_y"] == 1


NEAREST = ((5, 7, -2, 1), (4, 7, -10, 1))
WIDE, WIDE_TRUNC, WIDE_CLAMP = ((5, 7, 12, 0), (5, 10, 9, 0)), ((5, 4, 12, 0), (5, 10, 9, 0)), ((5, 7, 17, 0), (5, 10, 15, 0))


# FP32 carriers: how many workgroups of 64 x 64 are cut into 32 x 32 ones throughout; channels in multiples of 16, and pieces gathered from taps
@pytest.mark.parametrize("c,k,formats,planes,most", [(16, 3, WIDE, "ou", 512), (16, 3, WIDE_TRUNC, "ou", 512), (3, 3, WIDE, "ou", 384), (6, 3, WIDE, "ou", 384),
                                                     (20, 3, WIDE, "ou", 384), (3, 5, WIDE_TRUNC, "ou", 384)])
def test_small_fp32_recompute(rec, c, k, formats, planes, most):
    for blocks in (256, 257, 320, 321, 384, 385, 512, 513):
        M, N, name, p = conv(rec, 1, 64, blocks, c, 64, k, formats, planes)
        assert M == 64 * blocks and name == "launch_fast_bwd" and not p["packed"] and fits(M, N, p)
        assert (p["mix_tail"] == 2 * blocks * 2 and p["mix_main"] == 0) == (blocks <= most), (blocks, p)


# Filter rows of fewer than 16 codes and tensors of fewer run on FP32 carriers: on the tiles those kernels have
@pytest.mark.parametrize("formats", [PACKED, TRUNC])
@pytest.mark.parametrize("shape", [(1, 14, 14, 3, 64, 3), (8, 28, 28, 3, 128, 3), (4, 64, 64, 3, 64, 3), (2, 56, 56, 4, 64, 3), (5, 56, 56, 3, 64, 4), (1, 3, 2, 2, 40, 3)])
@pytest.mark.parametrize("planes", ["o", "ou", "u"])
def test_recompute_of_narrow_filters(rec, shape, planes, formats):
    M, N, name, p = conv(rec, *shape, formats, planes)
    assert name == "launch_fast_bwd" and not p["packed"] and fits(M, N, p)
    assert (p["tm"], p["tn"]) == (4, 4)                        # the only lane block of the FP32 recompute kernels' plain grids


@pytest.mark.parametrize("formats", [PACKED, TRUNC])
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("shape", [(1, 14, 14, 3, 64, 3), (4, 28, 28, 3, 64, 3), (3, 64, 64, 3, 64, 4), (12, 56, 56, 3, 64, 4), (8, 56, 57, 3, 128, 4), (1, 33, 33, 1, 64, 15)])
def test_forward_of_narrow_filters(rec, shape, order, formats):
    M, N, name, p = conv(rec, *shape, formats, None, order)
    small = -(-M // 32) * -(-N // 32) <= 128                   # 32 x 16 tiles throughout stay on packed carriers
    assert p["packed"] == small and not p["staged"] and fits(M, N, p)
    if small:
        assert p["mix_tail16"] and p["mix_main"] + p["mix_half"] == 0 and name == "launch_half_conv"
    else:
        assert name in ("launch_fast_conv", "launch_fast_amode", "launch_fast_in_mixed_seq", "launch_fast_in_mixed_chunk")


# widths that are no multiple of 32, whose small tiles write parts of cache lines: the blocks up to which tiles are 32 x 32, alone on their CUs or throughout
@pytest.mark.parametrize("N", [60, 64])
@pytest.mark.parametrize("formats,K,planes,order,most", [
    (PACKED, 160, "ou", 0, (320, 384)), (PACKED, 512, "ou", 0, (320, 384)), (PACKED, 768, "ou", 0, (320, 384)), (PACKED, 769, "ou", 0, (320, 384)), (PACKED, 513, "ou", 1, (192, 256)), (PACKED, 512, "ou", 1, (256, 256)),
    (PACKED, 255, "o", 0, (192, 192)), (PACKED, 256, "o", 0, (192, 320)), (PACKED, 1025, "o", 0, (192, 320)), (PACKED, 160, "o", 1, (256, 256)), (PACKED, 161, "o", 1, (192, 256)),
    (PACKED, 1024, "o", 1, (192, 256)), (PACKED, 1025, "o", 1, (192, 256)), (WIDE, 512, "ou", 0, (512, 512)), (WIDE, 513, "ou", 0, (512, 512)), (WIDE, 1025, "o", 0, (320, 384)), (WIDE, 1024, "o", 0, (384, 384)), (WIDE_TRUNC, 1025, "o", 0, (384, 384)), (WIDE, 96, "o", 0, (320, 320)),
    (TRUNC, 256, "ou", 0, (384, 384)), (TRUNC, 257, "ou", 0, (320, 384)), (NEAREST, 513, "ou", 0, (512, 512)), (NEAREST, 513, "o", 0, (384, 384))])
def test_partial_lines(rec, N, formats, K, planes, order, most):
    most = most[N == 64]
    for blocks in (1, 160, 161, 192, 193, 256, 257, 300, 301, 320, 321, 384, 385, 512, 513):
        M, qp, qa = 64 * blocks, lba_qfmt(*formats[0]), lba_qfmt(*formats[1])
        of, uf = BUF, BUF if "u" in planes else None
        rc = rec.lba_gemm_bwd_chunked(BUF, BUF, BUF, of, uf, of, uf, M, N, K, qp, qa, None) if order else rec.lba_gemm_bwd(BUF, BUF, BUF, of, uf, M, N, K, qp, qa, 0, None)
        name, p = taken(rec)
        assert rc == 0 and fits(M, N, p)
        small = p["tm"] == 2 if p["alone"] else p["mix_tail"] == 4 * blocks and p["mix_main"] == 0
        alone = 192 < blocks <= 256 and formats == PACKED and order == 0 and (planes == "o" or (K, N) == (769, 60))   # 64 x 64 ones alone on their CUs
        assert small == (blocks <= most and not alone), (blocks, name, p)


# tiles whose halves are empty count for what they hold
@pytest.mark.parametrize("N,formats,planes,blocks,small", [(32, WIDE, "o", 512, True), (32, WIDE, "ou", 1024, True), (32, WIDE, "ou", 1026, False), (32, PACKED, "o", 256, True),
                                                           (160, PACKED, "o", 228, True), (160, PACKED, "o", 300, True), (32, PACKED, "o", 384, True), (160, PACKED, "o", 234, False), (32, PACKED, "ou", 700, True), (160, PACKED, "ou", 384, True), (160, PACKED, "ou", 393, False), (160, WIDE, "ou", 510, True), (160, WIDE, "ou", 516, False), (64, PACKED, "o", 320, True), (64, PACKED, "o", 321, False), (70, WIDE, "o", 384, True), (70, WIDE, "o", 386, False), (70, WIDE_TRUNC, "o", 386, True), (70, WIDE_CLAMP, "o", 386, False), (32, WIDE, "o", 514, True)])
def test_empty_halves(rec, N, formats, planes, blocks, small):
    M = 64 * (blocks // -(-N // 64))
    assert rec.lba_gemm_bwd(BUF, BUF, BUF, BUF, BUF if "u" in planes else None, M, N, 700, lba_qfmt(*formats[0]), lba_qfmt(*formats[1]), 0, None) == 0
    name, p = taken(rec)
    assert (p["tm"] == 2 if p["alone"] else p["mix_tail"] > 0 and p["mix_main"] == 0) == small, (name, p)


# clamped products, chains of any length: small tiles on few workgroups
@pytest.mark.parametrize("rnd", [0, 1])
@pytest.mark.parametrize("K", [16, 64, 159, 160, 700])
def test_small_clamped_recompute(rec, K, rnd):
    for blocks, both, alone in [(1, True, True), (300, True, True), (400, True, False), (512, True, False), (768, False, False)]:
        for uf, small in ((BUF, both), (None, alone)):
            assert rec.lba_gemm_bwd(BUF, BUF, BUF, BUF, uf, 64 * blocks, 64, K, lba_qfmt(5, 7, 15, rnd), lba_qfmt(4, 7, 7, rnd), 0, None) == 0
            name, p = taken(rec)
            assert name == "launch_fast_bwd" and not p["packed"] and (p["mix_tail"] == 4 * blocks and p["mix_main"] == 0) == small, (blocks, uf)


# One plane or both: the plan is that of the planes asked for, from every entry point
@pytest.mark.parametrize("planes", ["o", "ou", "u"])
def test_planes_asked_for(rec, planes):
    of, uf = BUF if "o" in planes else None, BUF if "u" in planes else None
    alone = planes == "o"
    for fmt, (qp, qa), packed in [((4, 3, 7), PACKED, True), ((3, 4, 3), ((5, 7, 1, 0), (4, 7, 2, 0)), True), ((4, 3, 7), WIDE, False), ((3, 4, 3), ((5, 7, 1, 0), (5, 10, 5, 0)), False)]:
        for blocks in (200, 300, 340, 400, 500):
            rc = rec.lba_gemm_bwd_in(BUF, BUF, BUF, of, uf, 64 * blocks, 64, 500, lba_infmt(*fmt), lba_infmt(*fmt), lba_qfmt(*qp), lba_qfmt(*qa), 0, None)
            name, p = taken(rec)
            assert rc == 0 and p["of_only"] == alone and p["packed"] == packed and fits(64 * blocks, 64, p)
            # 32 x 32 throughout: FP32 up to 384 and 512, packed from 257 to 320 and with both planes to 384 (fewer: truncated products, others have kernels of their own)
            small = p["mix_tail"] == 4 * blocks and p["mix_main"] == 0
            trunc = fmt == (3, 4, 3)
            want = blocks <= (384 if alone else 512) if not packed else blocks <= (320 if alone else 384) and (trunc or blocks > 256)
            assert small == want, (blocks, p)
    for c, formats, packed in [(32, PACKED, True), (20, PACKED, True), (32, WIDE, False), (3, WIDE, False)]:
        _, _, name, p = conv(rec, 1, 64, 300, c, 64, 3, formats, planes)
        assert p["of_only"] == alone and p["packed"] == packed
        assert (p["mix_tail"] == 1200) == (not alone or c == 32)


# the overflow plane alone: whole taps up to 384, gathered rows up to 320 from two k-tiles on and up to 256 with truncated products
@pytest.mark.parametrize("c,k,formats,most", [(16, 3, WIDE, 384), (16, 3, WIDE_TRUNC, 384), (3, 5, WIDE, 320), (3, 3, WIDE, 256), (3, 5, WIDE_TRUNC, 256)])
def test_small_fp32_overflow_plane(rec, c, k, formats, most):
    for blocks in (256, 257, 320, 321, 384, 385):
        M, N, name, p = conv(rec, 1, 64, blocks, c, 64, k, formats, "o")
        assert name == "launch_fast_bwd" and p["of_only"] and fits(M, N, p)
        assert (p["mix_tail"] == 4 * blocks and p["mix_main"] == 0) == (blocks <= most), (blocks, p)


WIDE7, WIDE10 = ((5, 7, 12, 0), (5, 7, -2, 0)), ((5, 7, 12, 0), (5, 10, -2, 0))     # packed, sums beyond FP16's range


# 513 to 1024 workgroups of 64 x 64 (a batch, which has no tail): the finer block throughout on FP32 carriers, on packed ones where it saves half a round of 256
@pytest.mark.parametrize("batch", [512, 513, 640, 641, 768, 769, 896, 897, 1024, 1025])
def test_half_rounds(rec, batch):
    half_round = batch in (513, 640, 769, 896)
    for formats, K, order, half_rounds in [(PACKED, 768, 0, True), (PACKED, 32, 1, True), (PACKED, 771, 0, True), (PACKED, 17, 1, True), (NEAREST, 768, 0, False), (WIDE, 768, 0, False),
                                           (WIDE7, 96, 0, True), (WIDE7, 80, 0, False), (WIDE7, 256, 1, True), (WIDE7, 240, 1, False), (WIDE10, 96, 0, True), (WIDE10, 771, 0, False)]:
        rc = rec.lba_gemm_batched(BUF, BUF, BUF, batch, 64 * K, 64 * K, 64 * 64, 64, 64, K, lba_qfmt(*formats[0]), lba_qfmt(*formats[1]), order, None)
        name, p = taken(rec)
        assert rc == 0 and p["mix_tail"] == 0 and p["packed"] == (formats not in (NEAREST, WIDE)) and fits(64, 64, p)
        finer = 512 < batch <= 1024 and (half_round or not half_rounds)
        assert (p["tm"], p["tn"]) == ((2, 4) if finer else (4, 4)), (formats, K, order)


# im2col rows beyond FP16's range: gathered from several taps, and whole taps
@pytest.mark.parametrize("c,k,order,half_rounds", [(20, 2, 0, True), (20, 2, 1, True), (12, 2, 0, True), (16, 2, 0, False), (16, 3, 0, True), (16, 3, 1, False), (32, 3, 1, True)])
def test_wide_convolutions(rec, c, k, order, half_rounds):
    M, N, name, p = conv(rec, 1, 64 + (k == 2) * -1, 768 + (k == 2) * -1, c, 64, k, WIDE7, None, order)
    assert M == 64 * 768 and name == "launch_wide_conv" and p["mix_tail"] == 0 and fits(M, N, p)
    assert (p["tm"], p["tn"]) == ((4, 4) if half_rounds else (2, 4))


# members whose last rows fill half a tile of 64: the finer block has fewer rounds than twice the workgroups of 64 x 64
@pytest.mark.parametrize("batch,M,finer", [(64, 197, True), (60, 197, True), (48, 197, False), (36, 197, True), (384, 70, True), (256, 128, False), (500, 96, True), (340, 100, False), (700, 32, True)])
def test_half_tiles(rec, batch, M, finer):
    N = 197 if M == 197 else 64
    rc = rec.lba_gemm_batched(BUF, BUF, BUF, batch, M * 64, N * 64, M * N, M, N, 64, lba_qfmt(*PACKED[0]), lba_qfmt(*PACKED[1]), 0, None)
    name, p = taken(rec)
    blocks = batch * -(-M // 64) * -(-N // 64)
    assert rc == 0 and fits(M, N, p) and 512 < blocks <= 1024 or blocks == 512
    assert (p["tm"], p["tn"]) == ((2, 4) if finer else (4, 4)), blocks


# a tail of 32 x 32 tiles on 700 workgroups: M10E5 from 512 steps on, narrower accumulators not
@pytest.mark.parametrize("formats,K,tail", [(WIDE10, 512, True), (WIDE10, 496, False), (WIDE10, 64, False), (WIDE7, 2304, False), (PACKED, 2304, False), (WIDE, 768, True)])
def test_tail_of_a_last_round(rec, formats, K, tail):
    for order in (0, 1):
        assert rec.lba_gemm(BUF, BUF, BUF, 64 * 700, 64, K, lba_qfmt(*formats[0]), lba_qfmt(*formats[1]), order, None) == 0
        name, p = taken(rec)
        assert (p["mix_main"] == 512 and p["mix_tail"] == 752) == tail and (tail or p["mix_tail"] == 0)


# chunks of few outputs: side by side up to 64 workgroups of 32 x 32 (128 on short chains), one after the other with waves that stage beyond
@pytest.mark.parametrize("K,most", [(1712, 64), (224, 64), (208, 128)])
def test_chunks_side_by_side(rec, K, most):
    for b32 in (1, 64, 65, 96, 97, 128, 129, 300):
        assert rec.lba_gemm(BUF, BUF, BUF, 32 * b32, 32, K, lba_qfmt(*PACKED[0]), lba_qfmt(*PACKED[1]), 1, None) == 0
        name, p = taken(rec)
        assert (p["kpar"] > 0) == (b32 <= most or (K == 208 and b32 > 256)), b32
        assert name == ("launch_kpar" if p["kpar"] else "launch_half") and (p["kpar"] > 0 or p["staged"])

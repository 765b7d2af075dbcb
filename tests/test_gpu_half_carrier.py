"""The forward tile on packed FP16 carriers (csrc/lba_half.h): every result is the oracle's, bit for bit, at the edges of
the rule that admits a format (both sides of every line), of the tiles and of the k remainders."""
import itertools

import numpy as np
import pytest
import torch

from paper_2401_14110_amd import binding as lb

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bits(x):
    return np.ascontiguousarray(x).view(np.uint32)


def codes(rng, shape, lo=0, hi=15, E=4):
    """Random codes whose exponent field lies in [lo, hi] (of a format with E exponent bits), zeros among them."""
    m = 7 - E
    c = rng.integers(0, 256, size=shape, dtype=np.uint8)
    e = np.clip((c >> m) & ((1 << E) - 1), lo, min(hi, (1 << E) - 1)).astype(np.uint8)
    c = ((c & 0x80) | (e << m) | (c & ((1 << m) - 1))).astype(np.uint8)
    return np.where(rng.random(shape) < 0.2, np.uint8(0), c)


def product(A, B, qp, qa, order, fa=None, fb=None):
    dA, dB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    C = lb.gemm(dA, dB, qp, qa, order=order) if fa is None else lb.gemm_in(dA, dB, fa, fb, qp, qa, order=order)
    torch.cuda.synchronize()
    return C.cpu().numpy()


def slots(M, N, K, qp, qa):
    return lb.lba_plan_query(M, N, K, qp, qa, 0)["valu_per_mac_x100"]


@pytest.mark.parametrize("qae,qam", [(4, 1), (4, 7), (4, 10), (4, 11), (3, 4), (2, 3), (5, 7)])
def test_every_side_of_the_admission_rule(ref, qae, qam):
    # product domains from "the largest product is just too large" to "a scaled unit would fall below FP16's", and the
    # accumulator's domain moving past the product's on both sides (kc from 2^-25 to 2^16); M = 11 and E = 5 stay on FP32
    rng = np.random.default_rng(11)
    A, B = codes(rng, (48, 83)), codes(rng, (36, 83))
    packed = set()
    for bp, ba in itertools.product((13, 12, 11, 4, -1, -9, -14, -16, -17, -18), (16, 11, 7, -2, -9, -15, -17, -24)):
        qp, qa = (6, 7, bp, 0), (qae, qam, ba, 0)
        packed.add(slots(48, 36, 83, qp, qa) == 250)
        for order in (0, 1):
            got = product(A, B, qp, qa, order)
            want = ref.gemm(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order)
            assert np.array_equal(bits(got), bits(want)), (qp, qa, order)
    assert packed == ({False} if qam > 10 or qae > 4 else {True, False})


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 129, 200])
def test_k_remainders_and_ragged_tiles(ref, K):
    # quiet operands (clamp-free tiles) and loud ones (every sum saturates), rows and columns off the tiles of every region (the
    # chunked order's grids are too small for the packed tile here: lba_kpar_kernel from K = 17 on; the next test has larger ones)
    rng = np.random.default_rng(K)
    qp, qa = (5, 7, -1, 0), (4, 7, -9, 0)
    for (M, N), (lo, hi) in itertools.product([(33, 18), (65, 130), (300, 257)], [(0, 9), (3, 15)]):
        assert slots(M, N, K, qp, qa) == 250
        assert lb.lba_plan_kernel_name(M, N, K, qp, qa, 0).startswith("lba_half")
        assert lb.lba_plan_kernel_name(M, N, K, qp, qa, 1).startswith("lba_kpar" if K > 16 else "lba_half")
        A, B = codes(rng, (M, K), lo, hi), codes(rng, (N, K), lo, hi)
        for order in (0, 1):
            got = product(A, B, qp, qa, order)
            assert np.array_equal(bits(got), bits(ref.gemm(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order))), (M, N, K, lo, order)


@pytest.mark.parametrize("K", [1, 15, 17, 32, 33, 63, 65, 97, 129, 200])
@pytest.mark.parametrize("M,N,kernel", [(1040, 530, "lba_half_kernel<2, 4,"), (8200, 530, "lba_half_kernel<4, 4,"),
                                        (9000, 66, "lba_half_mixed_kernel"), (20000, 66, "lba_half_mixed_kernel"), (33000, 66, "lba_half_mixed_kernel")])
def test_k_remainders_of_the_chunked_packed_tile(ref, M, N, kernel, K):
    # chunks of 16 on grids of 512 workgroups of 32 x 32 and more: every lane block, and mixed grids with 48-row and 32 x 32 tails;
    # sampled rows of every region, short last chunks, quiet and loud operands
    rng = np.random.default_rng([M, K])
    qp, qa = (5, 7, -1, 0), (4, 7, -9, 0)
    name = lb.lba_plan_kernel_name(M, N, K, qp, qa, 1)
    assert name.startswith(kernel), name
    rows = np.array(sorted({0, 1, 63, 64, M // 2, M - 49, M - 33, M - 2, M - 1} | set(int(r) for r in rng.integers(0, M, 60))))
    for lo, hi in [(0, 9), (3, 15)]:
        A, B = codes(rng, (M, K), lo, hi), codes(rng, (N, K), lo, hi)
        got = product(A, B, qp, qa, 1)[rows]
        assert np.array_equal(bits(got), bits(ref.gemm(A[rows], B, ref.QFmt(*qp), ref.QFmt(*qa), order=1))), (lo, name)


@pytest.mark.parametrize("fa,fb", [((3, 4, 3), (3, 4, 3)), ((2, 5, 1), (3, 4, 5)), ((4, 3, 9), (2, 5, -2)), ((2, 5, 1), (2, 5, 1)), ((5, 2, 15), (3, 4, 3))])
def test_operand_formats(ref, fa, fb):
    # products of up to 12 bits, truncated by Q_prod (10 bits of mantissa at most on packed carriers) or kept; E = 5
    # operands stay on FP32
    rng = np.random.default_rng(5)
    for (M, N, K), qpm in itertools.product([(70, 50, 96), (33, 20, 147)], (4, 7, 10, 12)):
        A, B = codes(rng, (M, K), E=fa[0]), codes(rng, (N, K), E=fb[0])
        for bp, ba, order in itertools.product((0, 6, 12), (2, 7, 10), (0, 1)):
            qp, qa = (6, qpm, bp, 0), (4, 7, ba, 0)
            got = product(A, B, qp, qa, order, fa, fb)
            want = ref.gemm_in(A, B, ref.InFmt(*fa), ref.InFmt(*fb), ref.QFmt(*qp), ref.QFmt(*qa), order=order)
            assert np.array_equal(bits(got), bits(want)), (M, N, K, qp, qa, order)


@pytest.mark.parametrize("K", [96, 147])
def test_operand_formats_on_plain_grids(ref, K):
    # 64 x 64 workgroups throughout (512 of them): products kept, flushed and truncated; sampled rows, the tiles' edges among them
    rng = np.random.default_rng(K)
    M, N = 2048, 1024
    rows = np.array(sorted({0, 1, 63, 64, M - 1} | set(int(r) for r in rng.integers(0, M, 40))))
    for fa, fb in [((3, 4, 3), (3, 4, 3)), ((2, 5, 1), (3, 4, 5)), ((4, 3, 7), (3, 4, 3))]:
        A, B = codes(rng, (M, K), E=fa[0]), codes(rng, (N, K), E=fb[0])
        dA, dB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
        for (bp, qpm), order in itertools.product([(1, 4), (1, 7), (16, 12), (1, 12)], (0, 1)):
            qp, qa = (6, qpm, bp, 0), (4, 7, 2, 0)
            name = lb.lba_plan_kernel_name_in(M, N, K, fa, fb, qp, qa, order)
            assert name.startswith("lba_half_kernel<4, 4"), name
            C = lb.gemm_in(dA, dB, fa, fb, qp, qa, order=order)
            torch.cuda.synchronize()
            want = ref.gemm_in(A[rows], B, ref.InFmt(*fa), ref.InFmt(*fb), ref.QFmt(*qp), ref.QFmt(*qa), order=order)
            assert np.array_equal(bits(C.cpu().numpy()[rows]), bits(want)), (fa, fb, qp, order, name)


def planes(A, B, qp, qa, order):
    dA, dB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    got = lb.gemm_bwd_chunked(dA, dB, qp, qa) if order else lb.gemm_bwd(dA, dB, qp, qa)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in got]


@pytest.mark.parametrize("ba,bp,kernel,of_alone", [
    (2, 12, "lba_half_bwd", "lba_half_bwd"),       # kc = 2^-10: a product alone is FP16's smallest denormal number
    (1, 12, "lba_fast_bwd", "lba_half_bwd"),       # kc = 2^-11: FP32, but for the overflow plane alone
    (-9, 1, "lba_half_bwd", "lba_half_bwd"), (-10, 1, "lba_fast_bwd", "lba_half_bwd"),
    (-9, -1, "lba_half_bwd", "lba_half_bwd"), (10, 12, "lba_half_bwd", "lba_half_bwd"), (4, 11, "lba_half_bwd", "lba_half_bwd"),
    (3, 1, "lba_half_bwd", "lba_half_bwd"),
    (7, 15, "lba_fast_bwd", "lba_fast_bwd"), (7, 17, "lba_fast_bwd", "lba_fast_bwd"), (-2, -17, "lba_fast_bwd", "lba_fast_bwd"),   # products beyond FP16
    (7, 18, "lba_gen", "lba_gen"),                 # Q_prod cannot flush: the general kernel
])
def test_event_planes_on_both_sides_of_the_underflow_rule(ref, ba, bp, kernel, of_alone):
    # accumulators of 2 to 11 bits, operands full of subnormal codes and zeros, cancelling pairs next to R_UF
    rng = np.random.default_rng([ba + 100, bp + 100])
    for M, N, K in [(33, 18, 70), (70, 66, 97)]:
        A, B = codes(rng, (M, K), 0, 15), codes(rng, (N, K), 0, 15)
        A[:, 1::4] = A[:, 0::4][:, :A[:, 1::4].shape[1]] ^ 0x80      # x w, then almost -x w
        B[:, 1::4] = np.clip(B[:, 0::4][:, :B[:, 1::4].shape[1]].astype(np.int32) + rng.integers(-1, 2, B[:, 1::4].shape), 0, 255).astype(np.uint8)
        for qam, order in itertools.product((1, 7, 10), (0, 1)):
            qp, qa = (6, 7, bp, 0), (4, qam, ba, 0)
            assert lb.lba_plan_kernel_name(M, N, K, qp, qa, order, 1).startswith(kernel), order
            assert order or lb.lba_plan_kernel_name(M, N, K, qp, qa, order, 3).startswith(of_alone)
            got = planes(A, B, qp, qa, order)
            want = ref.gemm_bwd(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order, level2=True) if order else \
                ref.gemm_bwd(A, B, ref.QFmt(*qp), ref.QFmt(*qa))
            assert np.array_equal(bits(got[0]), bits(want[0])), (M, N, K, qp, qa, order)
            for i in range(1, len(want)):
                assert np.array_equal(got[i].view(np.uint32), want[i]), (M, N, K, qp, qa, order, "plane %d" % i)
            dA, dB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
            of = lb.gemm_bwd_chunked(dA, dB, qp, qa, want_c=False, want_uf=False)[1] if order else lb.gemm_bwd(dA, dB, qp, qa, want_c=False, want_uf=False)[1]
            torch.cuda.synchronize()
            assert np.array_equal(of.cpu().numpy().view(np.uint32), want[1]), (M, N, K, qp, qa, order, "overflow plane alone")


@pytest.mark.parametrize("K", [1, 15, 16, 17, 32, 33, 63, 65, 96, 129, 512, 530])
def test_event_planes_of_ragged_shapes(ref, K):
    # words at every remainder of k and of the second level, rows of the planes at every alignment, loud and quiet tiles, each
    # plane alone; saturated sums stay at R_OF beyond K and set no bit there
    rng = np.random.default_rng(K)
    qp, qa = (5, 7, -1, 0), (4, 7, -9, 0)
    for (M, N), (lo, hi) in itertools.product([(33, 17), (65, 66), (20, 131)], [(0, 9), (3, 15)]):
        A, B = codes(rng, (M, K), lo, hi), codes(rng, (N, K), lo, hi)
        for order in (0, 1):
            name = lb.lba_plan_kernel_name(M, N, K, qp, qa, order, 1)
            assert name.startswith("lba_half_bwd"), name
            want = ref.gemm_bwd(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order, level2=True) if order else \
                ref.gemm_bwd(A, B, ref.QFmt(*qp), ref.QFmt(*qa))
            got = planes(A, B, qp, qa, order)
            for i in range(len(want)):
                assert np.array_equal(bits(got[i]), bits(want[i])), (M, N, K, lo, order, i)
        dA, dB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
        _, of, _ = lb.gemm_bwd(dA, dB, qp, qa, want_c=False, want_uf=False)
        uf = torch.full((-(-K // 32), M, N), -1, dtype=torch.int32, device=DEV)
        assert lb.lba_gemm_bwd(dA.data_ptr(), dB.data_ptr(), None, None, uf.data_ptr(), M, N, K, qp, qa) == lb.OK
        torch.cuda.synchronize()
        w = ref.gemm_bwd(A, B, ref.QFmt(*qp), ref.QFmt(*qa))
        assert np.array_equal(bits(of.cpu().numpy()), bits(w[1])) and np.array_equal(bits(uf.cpu().numpy()), bits(w[2]))


def at(a, off):
    """A device copy of a that starts off bytes past a 16-byte boundary."""
    buf = torch.zeros(a.size + 32, dtype=torch.uint8, device=DEV)
    t = buf[off:off + a.size].view(a.shape)
    t.copy_(torch.from_numpy(a))
    return t


@pytest.mark.parametrize("n,h,w,c,cout,kh,kw,stride,pad", [
    (2, 9, 8, 5, 17, 3, 3, 1, 1),            # a filter row of 15 codes: byte by byte, on the smallest grids only
    (33, 28, 28, 5, 40, 3, 3, 1, 1),         # ... and on FP32 on any other
    (2, 9, 8, 16, 17, 3, 1, 1, 1),           # one tap to a filter row, aligned
    (2, 9, 8, 17, 18, 3, 1, 2, 2),           # a filter row one code longer than a piece
    (3, 11, 7, 3, 66, 7, 7, 2, 3),           # two filter rows to a piece, cut off at both edges of the image
    (1, 6, 5, 9, 130, 2, 2, 1, 4),           # padding wider than the image's reach: pieces wholly outside, before and after it
    (1, 4, 4, 1, 3, 3, 3, 1, 0),             # a tensor of exactly 16 bytes
    (1, 3, 5, 1, 3, 3, 3, 1, 1),             # one byte short of that
    (4, 40, 40, 6, 300, 3, 3, 1, 1),         # the large lane blocks
])
def test_pieces_of_im2col_rows(ref, n, h, w, c, cout, kh, kw, stride, pad):
    rng = np.random.default_rng([n, c, kw])
    qp, qa = (5, 7, -1, 0), (4, 7, -9, 0)
    X, W = codes(rng, (n, h, w, c)), codes(rng, (cout, kh, kw, c))
    B = W.reshape(cout, kh * kw * c)
    for (ox, ow), order in itertools.product([(0, 0), (1, 0), (0, 3), (13, 8)], (0, 1)):
        got = lb.conv2d(at(X, ox), at(W, ow), qp, qa, stride=stride, pad=pad, order=order)
        torch.cuda.synchronize()
        want = ref.gemm(ref.im2col_nhwc(X, kh, kw, stride, pad), B, ref.QFmt(*qp), ref.QFmt(*qa), order=order)
        assert np.array_equal(bits(got.cpu().numpy().reshape(want.shape)), bits(want)), (ox, ow, order)


@pytest.mark.parametrize("M,N,K", [(1, 1, 15), (1, 1, 16), (3, 5, 3), (1, 40, 16), (16, 1, 1), (33, 31, 48), (64, 64, 257),
                                   (1000, 700, 64), (1000, 700, 83)])
def test_pieces_of_rows_at_any_alignment(ref, M, N, K):
    # operands under 16 bytes stay on FP32; aligned and unaligned forms of the small and of the large lane blocks
    rng = np.random.default_rng([M, K])
    qp, qa = (5, 7, -1, 0), (4, 7, -9, 0)
    A, B = codes(rng, (M, K)), codes(rng, (N, K))
    assert (slots(M, N, K, qp, qa) == 250) == (M * K >= 16 and N * K >= 16)
    for (oa, ob), order in itertools.product([(0, 0), (1, 0), (0, 15), (4, 8)], (0, 1)):
        got = lb.gemm(at(A, oa), at(B, ob), qp, qa, order=order)
        torch.cuda.synchronize()
        assert np.array_equal(bits(got.cpu().numpy()), bits(ref.gemm(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order))), (oa, ob, order)


def test_rounded_products_of_im2col_rows(ref):
    # products that Q_prod truncates, on mixed grids and on a plain one (33 x 56 x 56 rows), aligned and not
    rng = np.random.default_rng(77)
    qp, qa = (5, 4, -1, 0), (4, 7, -9, 0)
    for n, h, w, c, cout in [(4, 40, 40, 16, 40), (4, 40, 40, 6, 40), (2, 9, 8, 16, 17), (33, 56, 56, 3, 64)]:
        X, W = codes(rng, (n, h, w, c)), codes(rng, (cout, 3, 3, c))
        got = lb.conv2d(at(X, 0), at(W, 0), qp, qa, stride=1, pad=1)
        torch.cuda.synchronize()
        want = ref.gemm(ref.im2col_nhwc(X, 3, 3, 1, 1), W.reshape(cout, 9 * c), ref.QFmt(*qp), ref.QFmt(*qa))
        assert np.array_equal(bits(got.cpu().numpy().reshape(want.shape)), bits(want)), (n, h, w, c, cout)

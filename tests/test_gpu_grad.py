"""GPU parity of the gradient side (lba_last_overflow, lba_grad) against the float64 gradient oracle.
Two bars: bit-exact where every FP32 product and partial sum is exactly representable (small dyadic g,
narrow operand range), and the derived FP32 bound  (terms + 1) * 2^-24 * sum|terms|  (times 2) on
general data, where the order of the summation is not fixed."""
import numpy as np
import pytest
import torch

from paper_2401_14110_amd import binding as lb

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
QP, QA = (5, 7, 15, 0), (4, 7, 7, 0)


@pytest.fixture(scope="module")
def gref(ref):
    from oracle import lba_grad_ref
    return lba_grad_ref


def codes(rng, shape, lo=0, hi=15):
    e = rng.integers(lo, hi + 1, shape); m = rng.integers(0, 8, shape); s = rng.integers(0, 2, shape)
    c = (s << 7) | (e << 3) | m
    return np.where((c & 0x7F) == 0x7F, c & 0xFE, c).astype(np.uint8)


def gpu_inputs(ref, A, B, qp, qa, order=0):
    tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    if order == 0:
        _, of, _ = lb.gemm_bwd(tA, tB, qp, qa, want_c=False)
    else:
        _, of, _, _, _ = lb.gemm_bwd_chunked(tA, tB, qp, qa, want_c=False)
    return tA, tB, of


def run_grad(tG, tA, tB, ste, of, K):
    last = lb.last_overflow(of, K) if ste == lb.STE_RECURSIVE_OF else None
    dX, dW = lb.grad(tG, tA, tB, ste, of_plane=of if ste == lb.STE_IMMEDIATE_OF else None, last_of=last)
    torch.cuda.synchronize()
    return dX.cpu().numpy(), dW.cpu().numpy()


def test_last_overflow_index(ref, gref):
    rng = np.random.default_rng(90)
    seen_some = seen_none = False
    for (M, N, K), lo, hi in [((70, 66, 100), 0, 15), ((33, 130, 64), 3, 12), ((5, 3, 31), 0, 15), ((64, 64, 1), 8, 15),
                              ((20, 24, 200), 2, 8)]:
        A = codes(rng, (M, K), lo, hi); B = codes(rng, (N, K), lo, hi)
        _, _, of = gpu_inputs(ref, A, B, QP, QA)
        got = lb.last_overflow(of, K)
        torch.cuda.synchronize()
        _, wof, _ = ref.gemm_bwd(A, B, ref.QFmt(*QP), ref.QFmt(*QA))
        want = gref.last_overflow(wof, K)
        assert np.array_equal(got.cpu().numpy(), want), (M, N, K)
        seen_some |= bool((want >= 0).any()); seen_none |= bool((want < 0).any())
    assert seen_some and seen_none


@pytest.mark.parametrize("ste", [0, 1, 2])
def test_exactly_representable_sums_are_bit_exact(ref, gref, ste):
    # g in {-2, ..., 2} in steps of 1/4 and operand values that are multiples of 2^-5 below 16: every term
    # and every partial sum is exact in FP32, so any summation order gives the oracle's value bit for bit.
    # Shapes: ragged rows and columns, K across the 64-lane and word boundaries, N % 4 != 0 (the general
    # path), tall M (the sum over m is split and combined with atomic adds).
    rng = np.random.default_rng(91 + ste)
    QP, QA = (4, 7, 12, 0), (4, 7, 10, 0)                          # R_OF = 63.75: these operands overflow often
    differs = 0
    for (M, N, K) in [(64, 64, 64), (70, 66, 100), (33, 130, 65), (5, 3, 31), (16, 4, 33), (3000, 24, 40), (40, 2100, 70)]:
        A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
        tA, tB, of = gpu_inputs(ref, A, B, QP, QA)
        dX, dW = run_grad(torch.from_numpy(G).to(DEV), tA, tB, ste, of, K)
        wX, wW = gref.grad(G, A, B, ref.QFmt(*QP), ref.QFmt(*QA), ste)
        assert np.array_equal(dX, wX.astype(np.float32)), (M, N, K, "dX", np.abs(dX - wX).max())
        assert np.array_equal(dW, wW.astype(np.float32)), (M, N, K, "dW", np.abs(dW - wW).max())
        iX, _ = gref.grad(G, A, B, ref.QFmt(*QP), ref.QFmt(*QA), 0)
        differs += int(not np.array_equal(wX, iX))
    assert differs == (0 if ste == 0 else 7)                        # every case has overflow events


@pytest.mark.parametrize("order", [0, 1])
def test_general_data_within_the_fp32_bound(ref, gref, order):
    rng = np.random.default_rng(95 + order)
    for (M, N, K), qp, qa in [((130, 70, 200), QP, QA), ((66, 300, 96), (4, 7, 9, 0), (4, 3, 7, 0)),
                              ((300, 64, 147), (5, 7, 15, 1), (4, 7, 7, 1))]:
        A = codes(rng, (M, K)); B = codes(rng, (N, K))
        G = rng.standard_normal((M, N)).astype(np.float32)
        tA, tB, of = gpu_inputs(ref, A, B, qp, qa, order)
        for ste in ((0, 1, 2) if order == 0 else (1,)):           # recursive: sequential order only
            dX, dW = run_grad(torch.from_numpy(G).to(DEV), tA, tB, ste, of, K)
            wX, wW = gref.grad(G, A, B, ref.QFmt(*qp), ref.QFmt(*qa), ste, order)
            aX, aW = gref.grad_abs(G, A, B, ref.QFmt(*qp), ref.QFmt(*qa), ste, order)
            tolX = 2 * (N + 1) * 2.0 ** -24 * aX + 1e-30
            tolW = 2 * (M + 1) * 2.0 ** -24 * aW + 1e-30
            assert (np.abs(dX - wX) <= tolX).all(), (M, N, K, ste, "dX", (np.abs(dX - wX) / tolX).max())
            assert (np.abs(dW - wW) <= tolW).all(), (M, N, K, ste, "dW", (np.abs(dW - wW) / tolW).max())


def test_immediate_estimator_with_the_diff_plane(ref, gref):
    # "Immediate / DIFF" (Sec. 4): the DIFF plane of lba_gemm_bwd_diff goes where the OF plane goes.
    rng = np.random.default_rng(99)
    QPd, QAd = (4, 7, 12, 0), (4, 7, 10, 0)
    for (M, N, K), order, eps2 in [((70, 66, 100), 0, 0.25), ((33, 130, 65), 1, 0.25), ((64, 24, 40), 0, 0.0)]:
        A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
        tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
        _, diff = lb.gemm_bwd_diff(tA, tB, QPd, QAd, eps2, order=order, want_c=False)
        dX, dW = lb.grad(torch.from_numpy(G).to(DEV), tA, tB, lb.STE_IMMEDIATE_OF, of_plane=diff)
        torch.cuda.synchronize()
        wX, wW = gref.grad(G, A, B, ref.QFmt(*QPd), ref.QFmt(*QAd), gref.STE_IMMEDIATE_DIFF, order,
                           c=gref.coefficients(A, B, ref.QFmt(*QPd), ref.QFmt(*QAd), gref.STE_IMMEDIATE_DIFF, order, eps2))
        assert np.array_equal(dX.cpu().numpy(), wX.astype(np.float32)), (M, N, K, "dX")
        assert np.array_equal(dW.cpu().numpy(), wW.astype(np.float32)), (M, N, K, "dW")
        oX, _ = gref.grad(G, A, B, ref.QFmt(*QPd), ref.QFmt(*QAd), gref.STE_IMMEDIATE_OF, order)
        assert not np.array_equal(wX, oX)                               # DIFF blocks more than overflow alone


def test_matrix_core_path_identity_and_recursive(ref, gref):
    # Shapes the dense (matrix-core) path takes (N % 4 == 0; K odd: groups of codes read out of two aligned words): ragged against its 128 x 128 tiles and
    # 32-deep steps, several k blocks, sums split over workgroups.  The recursive estimator gets last-overflow
    # indices written by hand: every position relative to the 128-blocks (first and last k of a block, K - 1,
    # none), so that the masked dense part and the sliver pass must meet exactly.  Bit-exact on data whose
    # sums are exactly representable, then the FP32 bound on general data.
    rng = np.random.default_rng(314)
    # (7300, 4, 2052): enough row tiles for the 128 x 256 variant of the dense kernel (256-wide k blocks)
    for (M, N, K) in [(130, 68, 260), (260, 132, 132), (64, 516, 640), (3000, 24, 40), (40, 2100, 72), (128, 128, 128),
                      (257, 36, 1028), (7300, 4, 2052), (1500, 64, 147), (70, 20, 1), (33, 8, 259)]:
        A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
        last = rng.integers(-1, K, (M, N)).astype(np.int32)
        edge = rng.integers(0, 8, (M, N))
        last = np.where(edge == 0, -1, last)
        last = np.where(edge == 1, K - 1, last)
        last = np.where(edge == 2, (last // 128) * 128, last)                     # first k of a block
        last = np.where(edge == 3, np.minimum((last // 128) * 128 + 127, K - 1), last)   # last k of a block
        tL = torch.from_numpy(last).to(DEV)
        c_rec = np.arange(K)[None, None, :] > last[:, :, None]
        for exact in (True, False):
            G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32) if exact else rng.standard_normal((M, N)).astype(np.float32)
            tG = torch.from_numpy(G).to(DEV)
            for ste, c in ((lb.STE_IDENTITY, None), (lb.STE_RECURSIVE_OF, c_rec)):
                dX, dW = lb.grad(tG, tA, tB, ste, last_of=tL if ste == lb.STE_RECURSIVE_OF else None)
                torch.cuda.synchronize()
                dX, dW = dX.cpu().numpy(), dW.cpu().numpy()
                cc = c if c is not None else np.ones((M, N, K), dtype=bool)
                wX, wW = gref.grad(G, A, B, None, None, ste, c=cc)
                if exact:
                    assert np.array_equal(dX, wX.astype(np.float32)), (M, N, K, ste, "dX", np.abs(dX - wX).max())
                    assert np.array_equal(dW, wW.astype(np.float32)), (M, N, K, ste, "dW", np.abs(dW - wW).max())
                else:
                    aX, aW = gref.grad_abs(G, A, B, None, None, ste, c=cc)
                    assert (np.abs(dX - wX) <= 2 * (N + 1) * 2.0 ** -24 * aX + 1e-30).all(), (M, N, K, ste, "dX")
                    assert (np.abs(dW - wW) <= 2 * (M + 1) * 2.0 ** -24 * aW + 1e-30).all(), (M, N, K, ste, "dW")
    # code matrices that start 1, 2 and 3 bytes off a 4-byte boundary (rows then start anywhere, also with K % 4 == 0):
    # the groups of four codes come out of the two aligned words around them; the last group of the last row ends
    # with the buffer
    for off, (M, N, K) in ((1, (140, 36, 260)), (2, (70, 132, 147)), (3, (300, 8, 129))):
        A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        bufA = torch.zeros(M * K + off, dtype=torch.uint8, device=DEV); bufA[off:] = torch.from_numpy(A).to(DEV).reshape(-1)
        bufB = torch.zeros(N * K + off, dtype=torch.uint8, device=DEV); bufB[off:] = torch.from_numpy(B).to(DEV).reshape(-1)
        tA, tB = bufA[off:].view(M, K), bufB[off:].view(N, K)
        assert tA.data_ptr() % 4 == off and tB.data_ptr() % 4 == off
        G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
        dX, dW = lb.grad(torch.from_numpy(G).to(DEV), tA, tB, lb.STE_IDENTITY)
        torch.cuda.synchronize()
        wX, wW = gref.grad(G, A, B, None, None, lb.STE_IDENTITY, c=np.ones((M, N, K), dtype=bool))
        assert np.array_equal(dX.cpu().numpy(), wX.astype(np.float32)) and np.array_equal(dW.cpu().numpy(), wW.astype(np.float32)), (off, M, N, K)
    # the split of an FP32 factor into three bfloat16 pieces is exact (as long as the pieces and the products stay
    # FP32 normals): one term per sum, so the product itself must come back
    g = np.array([[1.0 + 2.0 ** -23, -3.1415927, 2.0 ** -80 * 1.6180339, 2.0 ** -60 * (1 + 2.0 ** -12)],
                  [16777215.0, -1e30, 2.0 ** 100, 7.0]], dtype=np.float32)
    M, N, K = 2, 4, 8
    A = np.zeros((M, K), dtype=np.uint8); B = np.zeros((N, K), dtype=np.uint8)
    B[:, :] = np.array([0x38, 0x3C, 0xC1, 0x7E, 0x01, 0x08, 0xB9, 0x30], dtype=np.uint8)[None, :]
    for n in range(N):                                               # one non-zero g per output sum
        Gn = np.zeros_like(g); Gn[:, n] = g[:, n]
        dX, _ = lb.grad(torch.from_numpy(Gn).to(DEV), torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), lb.STE_IDENTITY)
        torch.cuda.synchronize()
        vals = np.array([ref.decode(int(c)) for c in B[n]], dtype=np.float64)
        want = (Gn[:, n].astype(np.float64)[:, None] * vals[None, :]).astype(np.float32)
        assert np.array_equal(dX.cpu().numpy(), want), n


def test_arguments_views_and_degenerate_sizes(ref, gref):
    rng = np.random.default_rng(99)
    M, N, K = 40, 36, 50
    A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
    G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
    tA, tB, of = gpu_inputs(ref, A, B, QP, QA)
    wX, wW = gref.grad(G, A, B, ref.QFmt(*QP), ref.QFmt(*QA), 1)
    # G at an address that is not 16-byte aligned: the general path
    buf = torch.zeros(M * N + 1, dtype=torch.float32, device=DEV)
    buf[1:] = torch.from_numpy(G).to(DEV).reshape(-1)
    tG = buf[1:].view(M, N)
    dX, dW = lb.grad(tG, tA, tB, 1, of_plane=of)
    torch.cuda.synchronize()
    assert np.array_equal(dX.cpu().numpy(), wX.astype(np.float32)) and np.array_equal(dW.cpu().numpy(), wW.astype(np.float32))
    # one output only
    tG = torch.from_numpy(G).to(DEV)
    dX, none = lb.grad(tG, tA, tB, 1, of_plane=of, want_dw=False)
    none2, dW = lb.grad(tG, tA, tB, 1, of_plane=of, want_dx=False)
    torch.cuda.synchronize()
    assert none is None and none2 is None
    assert np.array_equal(dX.cpu().numpy(), wX.astype(np.float32)) and np.array_equal(dW.cpu().numpy(), wW.astype(np.float32))
    # status codes; nothing runs on these
    g, a, b, o = tG.data_ptr(), tA.data_ptr(), tB.data_ptr(), of.data_ptr()
    x = torch.empty(M * K, dtype=torch.float32, device=DEV).data_ptr()
    assert lb.lba_grad(g, a, b, o, None, None, None, M, N, K, 1) == lb.ERR_NULL
    assert lb.lba_grad(g, a, b, None, None, x, None, M, N, K, 1) == lb.ERR_NULL          # immediate needs the plane
    assert lb.lba_grad(g, a, b, o, None, x, None, M, N, K, 2) == lb.ERR_NULL             # recursive needs last_of
    assert lb.lba_grad(None, a, b, o, None, x, None, M, N, K, 0) == lb.ERR_NULL
    assert lb.lba_grad(g, a, b, o, None, x, None, M, N, K, 7) == lb.ERR_UNSUPPORTED
    assert lb.lba_grad(g, a, b, o, None, x, None, -1, N, K, 0) == lb.ERR_SHAPE
    assert lb.lba_last_overflow(o, None, M, N, K) == lb.ERR_NULL
    # empty sums: N == 0 gives dX = 0
    dXz = torch.full((M, K), 7.0, dtype=torch.float32, device=DEV)
    assert lb.lba_grad(None, None, None, None, None, dXz.data_ptr(), None, M, 0, K, 0) == lb.OK
    torch.cuda.synchronize()
    assert (dXz == 0).all()
    assert lb.lba_grad(g, a, b, None, None, x, None, M, N, 0, 0) == lb.OK


def pack_plane(c):
    """bool [M, N, K] -> uint32 [ceil(K/32), M, N], bit k % 32 of word k // 32."""
    M, N, K = c.shape
    W = (K + 31) // 32
    pad = np.zeros((M, N, W * 32), dtype=np.uint64)
    pad[:, :, :K] = c
    words = (pad.reshape(M, N, W, 32) << np.arange(32, dtype=np.uint64)).sum(axis=3).astype(np.uint32)
    return np.ascontiguousarray(np.moveaxis(words, 2, 0))

def test_immediate_estimator_on_clean_and_nearly_clean_planes(ref, gref):
    # Steps of the plane (16 rows x 16 s x 64 k) without a blocked coefficient take plain multiply-adds.  OF planes
    # written by hand: no bit at all, a few scattered bits, a dense corner next to clean steps, and a set bit in the
    # last word only; K ragged against 64 and 32.  Bit-exact on exactly representable sums, the FP32 bound otherwise.
    rng = np.random.default_rng(271)
    # K = 80 and 208: rows of codes 16-byte aligned (the codes of a step go through LDS) with a ragged last k block
    for (M, N, K) in [(64, 64, 128), (80, 48, 200), (200, 36, 70), (48, 132, 33), (72, 64, 80), (40, 48, 208)]:
        A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
        for case in range(4):
            of = np.zeros((M, N, K), dtype=bool)
            if case == 1:
                of = rng.random((M, N, K)) < 2e-4
            elif case == 2:
                of[16:32, 16:32, :min(K, 64)] = rng.random((16, 16, min(K, 64))) < 0.5
                of[M - 1, N - 1, K - 1] = True
            elif case == 3:
                of[:, :, K - 1] = rng.random((M, N)) < 0.1
            c = ~of
            tP = torch.from_numpy(pack_plane(of).view(np.int32)).to(DEV)
            for exact in (True, False):
                G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32) if exact else rng.standard_normal((M, N)).astype(np.float32)
                tG = torch.from_numpy(G).to(DEV)
                dX, dW = lb.grad(tG, tA, tB, lb.STE_IMMEDIATE_OF, of_plane=tP)
                torch.cuda.synchronize()
                dX, dW = dX.cpu().numpy(), dW.cpu().numpy()
                wX, wW = gref.grad(G, A, B, None, None, lb.STE_IMMEDIATE_OF, c=c)
                if exact:
                    assert np.array_equal(dX, wX.astype(np.float32)), (M, N, K, case, "dX")
                    assert np.array_equal(dW, wW.astype(np.float32)), (M, N, K, case, "dW")
                else:
                    aX, aW = gref.grad_abs(G, A, B, None, None, lb.STE_IMMEDIATE_OF, c=c)
                    assert (np.abs(dX - wX) <= 2 * (N + 1) * 2.0 ** -24 * aX + 1e-30).all(), (M, N, K, case, "dX")
                    assert (np.abs(dW - wW) <= 2 * (M + 1) * 2.0 ** -24 * aW + 1e-30).all(), (M, N, K, case, "dW")
                # the coefficient plane itself (bits taken as they are) gives the same products
                cX, cW = lb.grad(tG, tA, tB, lb.STE_COEF_PLANE, of_plane=torch.from_numpy(pack_plane(c).view(np.int32)).to(DEV))
                torch.cuda.synchronize()
                if exact:
                    assert np.array_equal(cX.cpu().numpy(), dX) and np.array_equal(cW.cpu().numpy(), dW), (M, N, K, case)


def test_coefficient_planes_and_the_recursive_estimator_of_the_chunked_order(ref, gref):
    rng = np.random.default_rng(97)
    QP2, QA2 = (4, 7, 12, 0), (4, 7, 10, 0)
    for (M, N, K) in [(64, 64, 64), (37, 68, 530), (70, 66, 100), (5, 3, 31), (16, 24, 1100)]:
        A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
        tA, tB, tG = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), torch.from_numpy(G).to(DEV)
        for order in (0, 1):
            if order == 0:
                _, of, _ = lb.gemm_bwd(tA, tB, QP2, QA2, want_c=False, want_uf=False)
                of2 = None
            else:
                _, of, _, of2, _ = lb.gemm_bwd_chunked(tA, tB, QP2, QA2, want_c=False, want_uf=False)
            for ste in (lb.STE_IMMEDIATE_OF, lb.STE_RECURSIVE_OF):
                coef = lb.ste_plane(of, K, ste, order, of2)
                torch.cuda.synchronize()
                want_c = gref.coefficients(A, B, ref.QFmt(*QP2), ref.QFmt(*QA2), ste, order)
                assert np.array_equal(coef.cpu().numpy().view(np.uint32), pack_plane(want_c)), (M, N, K, order, ste)
                assert 0 < want_c.sum() < want_c.size
                dX, dW = lb.grad(tG, tA, tB, lb.STE_COEF_PLANE, of_plane=coef)
                torch.cuda.synchronize()
                wX, wW = gref.grad(G, A, B, ref.QFmt(*QP2), ref.QFmt(*QA2), ste, order)
                assert np.array_equal(dX.cpu().numpy(), wX.astype(np.float32)), (M, N, K, order, ste, "dX")
                assert np.array_equal(dW.cpu().numpy(), wW.astype(np.float32)), (M, N, K, order, ste, "dW")
            # in place
            keep = lb.ste_plane(of, K, lb.STE_RECURSIVE_OF, order, of2).cpu()
            assert lb.lba_ste_plane(of.data_ptr(), of2.data_ptr() if of2 is not None else None, of.data_ptr(),
                                    M, N, K, lb.STE_RECURSIVE_OF, order) == lb.OK
            torch.cuda.synchronize()
            assert torch.equal(of.cpu(), keep)
    assert lb.lba_ste_plane(of.data_ptr(), None, of.data_ptr(), M, N, K, lb.STE_RECURSIVE_OF, 1) == lb.ERR_NULL
    assert lb.lba_ste_plane(of.data_ptr(), None, of.data_ptr(), M, N, K, lb.STE_IDENTITY, 0) == lb.ERR_UNSUPPORTED
    assert lb.lba_ste_plane(None, None, of.data_ptr(), M, N, K, lb.STE_IMMEDIATE_OF, 0) == lb.ERR_NULL


def test_immediate_estimator_split_by_bricks(ref, gref):
    # lba_grad_ws: bricks (128 rows x 32 summed indices x 256 k) without a blocked coefficient run on the matrix
    # cores, the others in the vector kernel; every term is added by exactly one of them.  Planes without any
    # overflow, with overflows in the last part of the chains only (clean and marked bricks side by side, in both
    # directions), and with overflows everywhere; shapes ragged against the bricks, several k bricks, sums split over
    # workgroups, the general path (N % 4 != 0: no bricks); a coefficient plane (recursive estimator of the chunked
    # order).  Bit-exact on exactly representable sums, then the FP32 bound on general data; the workspace is filled
    # with garbage first and is shared by consecutive calls.
    rng = np.random.default_rng(777)
    QPb, QAb = (4, 7, 12, 0), (4, 7, 10, 0)                        # R_OF = 63.75
    ws = torch.full((1 << 20,), 0xA5, dtype=torch.uint8, device=DEV)
    kinds = set()
    for (M, N, K), loud in [((300, 200, 600), "tail"), ((130, 68, 260), "none"), ((260, 132, 515), "all"), ((64, 516, 640), "tail"),
                            ((3000, 24, 300), "tail"), ((40, 2100, 72), "all"), ((257, 36, 1028), "tail"), ((70, 66, 100), "tail"),
                            ((33, 130, 65), "all"), ((1500, 64, 147), "rows")]:
        assert lb.lba_grad_workspace_bytes(M, N, K) <= ws.numel()
        A = codes(rng, (M, K), 2, 5); B = codes(rng, (N, K), 2, 5)           # products below 2^-5: no sum reaches R_OF
        if loud == "tail":
            A[:, K - K // 3:] = codes(rng, (M, K // 3), 6, 10); B[:, K - K // 3:] = codes(rng, (N, K // 3), 6, 10)
        elif loud == "all":
            A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        elif loud == "rows":
            A[M // 2: M // 2 + 40] = codes(rng, (40, K), 7, 10); B[:, :] = codes(rng, (N, K), 5, 8)
        tA, tB, of = gpu_inputs(ref, A, B, QPb, QAb)
        ofn = of.cpu().numpy()
        kinds.add("clean" if not ofn.any() else ("mixed" if (ofn == 0).all(axis=(1, 2)).any() or loud == "rows" else "dirty"))
        for exact in (True, False):
            G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32) if exact else rng.standard_normal((M, N)).astype(np.float32)
            if not exact:                                                    # general data: full-range operands in the loud part
                pass
            tG = torch.from_numpy(G).to(DEV)
            dX, dW = lb.grad(tG, tA, tB, lb.STE_IMMEDIATE_OF, of_plane=of, workspace=ws)
            torch.cuda.synchronize()
            dX, dW = dX.cpu().numpy(), dW.cpu().numpy()
            wX, wW = gref.grad(G, A, B, ref.QFmt(*QPb), ref.QFmt(*QAb), 1)
            if exact:
                assert np.array_equal(dX, wX.astype(np.float32)), (M, N, K, loud, "dX", np.abs(dX - wX).max())
                assert np.array_equal(dW, wW.astype(np.float32)), (M, N, K, loud, "dW", np.abs(dW - wW).max())
            else:
                aX, aW = gref.grad_abs(G, A, B, ref.QFmt(*QPb), ref.QFmt(*QAb), 1)
                assert (np.abs(dX - wX) <= 2 * (N + 1) * 2.0 ** -24 * aX + 1e-30).all(), (M, N, K, loud, "dX")
                assert (np.abs(dW - wW) <= 2 * (M + 1) * 2.0 ** -24 * aW + 1e-30).all(), (M, N, K, loud, "dW")
            # the same call without the workspace agrees within the same bound (bit for bit on exact data)
            pX, pW = lb.grad(tG, tA, tB, lb.STE_IMMEDIATE_OF, of_plane=of)
            torch.cuda.synchronize()
            if exact:
                assert np.array_equal(pX.cpu().numpy(), dX) and np.array_equal(pW.cpu().numpy(), dW)
    assert kinds == {"clean", "mixed", "dirty"}, kinds
    # a coefficient plane: the recursive estimator of the chunked order
    M, N, K = 260, 132, 515
    A = codes(rng, (M, K), 2, 5); B = codes(rng, (N, K), 2, 5)
    A[:, 300:400] = codes(rng, (M, 100), 6, 10); B[:, 300:400] = codes(rng, (N, 100), 6, 10)
    tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    _, of, _, of2, _ = lb.gemm_bwd_chunked(tA, tB, QPb, QAb, want_c=False)
    coef = lb.ste_plane(of, K, lb.STE_RECURSIVE_OF, order=1, of_plane2=of2)
    G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
    dX, dW = lb.grad(torch.from_numpy(G).to(DEV), tA, tB, lb.STE_COEF_PLANE, of_plane=coef, workspace=ws)
    torch.cuda.synchronize()
    wX, wW = gref.grad(G, A, B, ref.QFmt(*QPb), ref.QFmt(*QAb), 2, 1)
    assert np.array_equal(dX.cpu().numpy(), wX.astype(np.float32)) and np.array_equal(dW.cpu().numpy(), wW.astype(np.float32))
    c = gref.coefficients(A, B, ref.QFmt(*QPb), ref.QFmt(*QAb), 2, 1)
    assert 0 < c.sum() < c.size
    # argument errors: nothing is enqueued
    ptr = lambda t: t.data_ptr()
    args = (ptr(torch.from_numpy(G).to(DEV)), ptr(tA), ptr(tB), ptr(coef), None, ptr(dX), ptr(dW), M, N, K, lb.STE_COEF_PLANE)
    assert lb.lba_grad_ws(*args, None, 1 << 20) == lb.ERR_NULL
    assert lb.lba_grad_ws(*args, ptr(ws) + 4, 1 << 19) == lb.ERR_ALIGN
    assert lb.lba_grad_ws(*args, ptr(ws), lb.lba_grad_workspace_bytes(M, N, K) - 1) == lb.ERR_SHAPE
    assert lb.lba_grad_ws(*args, ptr(ws), lb.lba_grad_workspace_bytes(M, N, K)) == lb.OK
    torch.cuda.synchronize()


def brick_maps_of(ofn, M, N, K):
    """The two byte maps as the library lays them out (dX side first, each padded to 256 bytes), from an OF plane."""
    W = (K + 31) // 32
    words = ofn.view(np.uint32).copy()
    if K % 32:
        words[W - 1] &= np.uint32((1 << (K % 32)) - 1)
    nz = words != 0                                                          # [W, M, N]
    kb = (K + 255) // 256
    dx = np.zeros((kb, (M + 127) // 128, (N + 31) // 32), np.uint8)
    dw = np.zeros((kb, (N + 127) // 128, (M + 31) // 32), np.uint8)
    w, m, n = np.nonzero(nz)
    dx[w // 8, m // 128, n // 32] = 1
    dw[w // 8, n // 128, m // 32] = 1
    pad = lambda a: np.concatenate([a.ravel(), np.zeros((-a.size) % 256, np.uint8)])
    return np.concatenate([pad(dx), pad(dw)])


def test_recompute_call_leaves_the_brick_maps(ref, gref):
    # lba_gemm_bwd_ws + lba_grad_premapped: same C and planes as lba_gemm_bwd; the maps in the workspace are those of
    # the plane (computed here from the plane itself), whichever kernel wrote it: the scaled-domain kernel that marks
    # bricks as it goes (floor and nearest-even, both planes or the overflow plane alone, plain and mixed grids), or the
    # general kernel followed by the pass over the plane (any width).  Then the gradients from those maps against the oracle.
    rng = np.random.default_rng(4242)
    QPb, QAb = (4, 7, 12), (4, 7, 10)                                        # R_OF = 63.75
    GEN_P, GEN_A = (5, 3, 12), (4, 7, 10)                                    # Q_prod rounds the mantissa: general kernel with planes
    ws = torch.full((1 << 20,), 0x5A, dtype=torch.uint8, device=DEV)
    seen = set()
    cases = [((300, 200, 600), "tail", 0, True), ((130, 68, 260), "none", 0, True), ((260, 132, 515), "all", 1, True),
             ((64 * 392, 64, 72), "rows", 0, True), ((64 * 150 + 33, 132, 300), "tail", 0, False), ((257, 36, 1028), "tail", 1, False),
             ((70, 66, 100), "tail", 0, True), ((33, 130, 65), "all", 1, True), ((1500, 64, 147), "rows", 0, True),
             ((64 * 330, 64, 72), "rows", 0, False), ((64 * 330 + 5, 62, 65), "rows", 0, False)]
    for (M, N, K), loud, rnd, want_uf in cases:
        need = lb.lba_grad_workspace_bytes(M, N, K)
        assert 0 < need <= ws.numel()
        A = codes(rng, (M, K), 2, 5); B = codes(rng, (N, K), 2, 5)
        if loud == "tail":
            A[:, K - K // 3:] = codes(rng, (M, K // 3), 6, 10); B[:, K - K // 3:] = codes(rng, (N, K // 3), 6, 10)
        elif loud == "all":
            A = codes(rng, (M, K), 5, 10); B = codes(rng, (N, K), 5, 10)
        elif loud == "rows":
            A[M // 2: M // 2 + 40] = codes(rng, (40, K), 7, 10); B[:, :] = codes(rng, (N, K), 5, 8)
        tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
        for qp, qa in ((QPb, QAb), (GEN_P, GEN_A)):
            qpf, qaf = qp + (rnd,), qa + (rnd,)
            plan = lb.lba_plan_query(M, N, K, qpf, qaf, 0, 1 if want_uf else 3)
            C0, of0, uf0 = lb.gemm_bwd(tA, tB, qpf, qaf, want_uf=want_uf)
            ws.fill_(0x5A)
            C1, of1, uf1, _ = lb.gemm_bwd_ws(tA, tB, qpf, qaf, workspace=ws, want_uf=want_uf)
            torch.cuda.synchronize()
            assert torch.equal(C0.view(torch.int32), C1.view(torch.int32)) and torch.equal(of0, of1)
            assert (uf0 is None and uf1 is None) or torch.equal(uf0, uf1)
            got = ws[:need].cpu().numpy()
            want = brick_maps_of(of1.cpu().numpy(), M, N, K)
            assert want.size == need
            assert np.array_equal(got != 0, want != 0), (M, N, K, qp, rnd, plan["kernel"], int((got != 0).sum()), int(want.sum()))
            seen.add(("general" if plan["kernel"] == 1 else "fused") + ("+mixed" if plan["tail_blocks"] + plan["mid_blocks"] > 0 else "") +
                     ("+ragged" if N % 4 != 0 else ""))
            kb = (K + 255) // 256
            bricks = kb * (((M + 127) // 128) * ((N + 31) // 32) + ((N + 127) // 128) * ((M + 31) // 32))
            seen.add("clean" if not want.any() else ("dirty" if int(want.sum()) == bricks else "partly"))
            if qp is GEN_P and (M, N, K) != (300, 200, 600):
                continue                                                     # gradients: once per shape, and once on the general kernel's plane
            G = rng.standard_normal((M, N)).astype(np.float32)
            tG = torch.from_numpy(G).to(DEV)
            dX, dW = lb.grad_premapped(tG, tA, tB, of1, ws)
            torch.cuda.synchronize()
            dX, dW = dX.cpu().numpy(), dW.cpu().numpy()
            wX, wW = gref.grad(G, A, B, ref.QFmt(*qpf), ref.QFmt(*qaf), 1)
            aX, aW = gref.grad_abs(G, A, B, ref.QFmt(*qpf), ref.QFmt(*qaf), 1)
            assert (np.abs(dX - wX) <= 2 * (N + 1) * 2.0 ** -24 * aX + 1e-30).all(), (M, N, K, loud, "dX")
            assert (np.abs(dW - wW) <= 2 * (M + 1) * 2.0 ** -24 * aW + 1e-30).all(), (M, N, K, loud, "dW")
    assert {"fused", "fused+mixed", "general", "general+ragged", "fused+ragged", "clean", "dirty", "partly"} <= seen, seen


@pytest.mark.parametrize("M,N,K", [(70, 66, 100), (130, 64, 300)])
def test_a_plane_off_a_16_byte_boundary_marks_every_brick(ref, gref, M, N, K):
    # the general kernel's plane where the pass over it does not run: every brick is marked, and the gradients are the oracle's
    rng = np.random.default_rng(M)
    qp, qa = (5, 3, 12, 0), (4, 7, 10, 1)                                    # a rounded product and a nearest-even sum: the general kernel
    A = codes(rng, (M, K), 4, 9); B = codes(rng, (N, K), 4, 9)
    tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    assert lb.lba_plan_query(M, N, K, qp, qa, 0, 3)["kernel"] == 1
    words = lb.lba_mask_words(M, N, K)
    of = torch.empty(words + 4, dtype=torch.int32, device=DEV)[1:1 + words]
    assert of.data_ptr() % 16 == 4
    need = lb.lba_grad_workspace_bytes(M, N, K)
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device=DEV)
    assert lb.lba_gemm_bwd_ws(tA.data_ptr(), tB.data_ptr(), None, of.data_ptr(), None, M, N, K, qp, qa, ws.data_ptr(), need) == lb.OK
    torch.cuda.synchronize()
    assert bool((ws == 1).all())
    _, wof, _ = ref.gemm_bwd(A, B, ref.QFmt(*qp), ref.QFmt(*qa))
    assert wof.any() and np.array_equal(of.cpu().numpy().view(np.uint32).reshape(wof.shape), wof)
    G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
    tG = torch.from_numpy(G).to(DEV)
    dX, dW = torch.empty(M, K, device=DEV), torch.empty(N, K, device=DEV)
    assert lb.lba_grad_premapped(tG.data_ptr(), tA.data_ptr(), tB.data_ptr(), of.data_ptr(), dX.data_ptr(), dW.data_ptr(), M, N, K,
                                 ws.data_ptr(), need) == lb.OK
    torch.cuda.synchronize()
    wX, wW = gref.grad(G, A, B, ref.QFmt(*qp), ref.QFmt(*qa), 1)
    aX, aW = gref.grad_abs(G, A, B, ref.QFmt(*qp), ref.QFmt(*qa), 1)
    assert (np.abs(dX.cpu().numpy() - wX) <= 2 * (N + 1) * 2.0 ** -24 * aX + 1e-30).all()
    assert (np.abs(dW.cpu().numpy() - wW) <= 2 * (M + 1) * 2.0 ** -24 * aW + 1e-30).all()


def test_split_sums_combined_in_the_workspace(ref, gref):
    # lba_grad_ws with lba_grad_workspace_bytes_fast bytes: where the matrix-core kernel cuts a sum over m or n across
    # workgroups, the slices are stored behind the maps and added in a fixed order instead of meeting in atomic adds.
    # All three estimators, both products split (few output tiles, long sums), rows of codes aligned and not; bit-exact
    # against the oracle on exactly representable sums; on general data the FP32 bound, for the identity estimator (no
    # atomic add left anywhere) the same bits on every call, and a workspace between the two sizes (some slices fit, or none) still gives correct sums.
    rng = np.random.default_rng(778)
    QPb, QAb = (4, 7, 12, 0), (4, 7, 10, 0)
    ptr = lambda t: t.data_ptr() if t is not None else None
    for (M, N, K) in [(300, 200, 600), (3000, 24, 300), (40, 2100, 72), (1500, 64, 147), (2600, 132, 128), (32, 28, 260)]:
        small, fast = lb.lba_grad_workspace_bytes(M, N, K), lb.lba_grad_workspace_bytes_fast(M, N, K)
        assert fast % 256 == 0 and fast >= small
        assert (fast > small) == ((M, N, K) != (32, 28, 260)), (M, N, K, small, fast)   # the last shape splits nothing
        A = codes(rng, (M, K), 2, 5); B = codes(rng, (N, K), 2, 5)
        A[:, K - K // 3:] = codes(rng, (M, K // 3), 6, 10); B[:, K - K // 3:] = codes(rng, (N, K // 3), 6, 10)   # overflows in the last third
        tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
        _, of, _ = lb.gemm_bwd(tA, tB, QPb, QAb, want_c=False)
        last = lb.last_overflow(of, K)
        assert bool((of != 0).any())
        qp, qa = ref.QFmt(*QPb), ref.QFmt(*QAb)
        ws = torch.full((fast,), 0x5A, dtype=torch.uint8, device=DEV)
        for exact in (True, False):
            G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32) if exact else rng.standard_normal((M, N)).astype(np.float32)
            tG = torch.from_numpy(G).to(DEV)
            for ste, kw in ((lb.STE_IDENTITY, {}), (lb.STE_RECURSIVE_OF, dict(last_of=last)), (lb.STE_IMMEDIATE_OF, dict(of_plane=of))):
                wX, wW = gref.grad(G, A, B, qp, qa, ste)
                outs = []
                for w in (ws, ws[:small + 256 * ((fast - small) // 512)], ws):      # all slices fit; the smaller product's or none; again
                    dX, dW = lb.grad(tG, tA, tB, ste, workspace=w, **kw)
                    torch.cuda.synchronize()
                    outs.append((dX.cpu().numpy(), dW.cpu().numpy()))
                if ste == lb.STE_IDENTITY:                                  # no atomic add anywhere: the same bits on every call
                    assert np.array_equal(outs[0][0], outs[2][0]) and np.array_equal(outs[0][1], outs[2][1]), (M, N, K, ste)
                for dX, dW in outs[:2]:
                    if exact:
                        assert np.array_equal(dX, wX.astype(np.float32)) and np.array_equal(dW, wW.astype(np.float32)), (M, N, K, ste)
                    else:
                        aX, aW = gref.grad_abs(G, A, B, qp, qa, ste)
                        assert (np.abs(dX - wX) <= 2 * (N + 1) * 2.0 ** -24 * aX + 1e-30).all(), (M, N, K, ste, "dX")
                        assert (np.abs(dW - wW) <= 2 * (M + 1) * 2.0 ** -24 * aW + 1e-30).all(), (M, N, K, ste, "dW")
    assert lb.lba_grad_workspace_bytes_fast(0, 8, 8) == 0 and lb.lba_grad_workspace_bytes_fast(1 << 31, 8, 8) == 0
    assert lb.lba_grad_workspace_bytes_fast(4096, 4096, 4096) == lb.lba_grad_workspace_bytes(4096, 4096, 4096)


@pytest.mark.parametrize("M,N,K", [(300, 201, 600), (131, 70, 257), (64, 515, 640), (1500, 63, 147), (129, 1, 300), (1, 130, 72),
                                   (33, 3, 31), (257, 37, 1028)])
@pytest.mark.parametrize("offset", [0, 1])
def test_any_width_and_alignment_on_the_matrix_cores(ref, gref, M, N, K, offset):
    # N % 4 != 0 and G off a 16-byte boundary: the identity estimator and the clean bricks of a plane whose rows are not
    # whole 16-byte groups (plane sizes of 0 to 3 words beyond the last group); clean and marked bricks side by side.
    # Sums of eighths below 2^24 units: exact in any order.
    rng = np.random.default_rng(M * 1000 + N)
    qp, qa = (4, 7, 12, 0), (4, 7, 10, 0)
    A = codes(rng, (M, K), 2, 5); B = codes(rng, (N, K), 2, 5)
    A[:, K - K // 3:] = codes(rng, (M, K // 3), 6, 10); B[N // 2:, K - K // 3:] = codes(rng, (N - N // 2, K // 3), 6, 10)
    tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    _, of, _ = lb.gemm_bwd(tA, tB, qp, qa, want_c=False)
    G = (rng.integers(-8, 9, (M, N)) / 4.0).astype(np.float32)
    flat = torch.zeros(M * N + 4, dtype=torch.float32, device=DEV)
    tG = flat[offset:offset + M * N].view(M, N)
    tG.copy_(torch.from_numpy(G))
    ws = torch.full((max(256, lb.lba_grad_workspace_bytes_fast(M, N, K)),), 0x5A, dtype=torch.uint8, device=DEV)
    coef = lb.ste_plane(of, K, lb.STE_RECURSIVE_OF)
    for ste, plane, est in ((lb.STE_IDENTITY, None, 0), (lb.STE_IMMEDIATE_OF, of, 1), (lb.STE_COEF_PLANE, coef, 2)):
        wX, wW = gref.grad(G, A, B, ref.QFmt(*qp), ref.QFmt(*qa), est)
        for w in (ws, ws[:max(256, lb.lba_grad_workspace_bytes(M, N, K))], None):
            dX, dW = lb.grad(tG, tA, tB, ste, of_plane=plane, workspace=w)
            torch.cuda.synchronize()
            assert np.array_equal(dX.cpu().numpy(), wX.astype(np.float32)), (ste, w is None, "dX")
            assert np.array_equal(dW.cpu().numpy(), wW.astype(np.float32)), (ste, w is None, "dW")


@pytest.mark.parametrize("M,N,K", [(40, 37, 70), (300, 201, 600), (131, 70, 257), (37, 515, 260)])
@pytest.mark.parametrize("what", ["tiny", "mixed", "infinite"])
def test_any_width_keeps_the_range_of_fp32(ref, gref, M, N, K, what):
    # Widths that are no multiple of 4 split g into bfloat16 pieces too; a step whose g do not split exactly (infinities, NaN,
    # values whose pieces would fall below FP32's normal range) runs in FP32.  tiny: all of G around 2^-118, whose last two
    # pieces are denormal numbers; mixed: some of them zero or of ordinary size; infinite: a few infinities and one NaN among
    # ordinary values, which reach their own row of dX and column of dW and nothing else.
    # Bound: 2 (terms + 1) 2^-24 sum|terms| as elsewhere in this file, and 2^-126 a term for results flushed as denormal.
    rng = np.random.default_rng([M, N, len(what)])
    qp, qa = (4, 7, 12, 0), (4, 7, 10, 0)
    A = codes(rng, (M, K), 2, 5); B = codes(rng, (N, K), 2, 5)
    A[:, K - K // 3:] = codes(rng, (M, K // 3), 6, 10); B[N // 2:, K - K // 3:] = codes(rng, (N - N // 2, K // 3), 6, 10)
    tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    _, of, _ = lb.gemm_bwd(tA, tB, qp, qa, want_c=False)
    coef = lb.ste_plane(of, K, lb.STE_RECURSIVE_OF)
    G = rng.standard_normal((M, N)).astype(np.float32)
    G = np.where(np.abs(G) < 2.0 ** -8, np.float32(2.0 ** -8), G)     # (times 2^-118: the smallest normal number)
    if what == "tiny":
        G *= np.float32(2.0 ** -118)
    elif what == "mixed":
        G[rng.random((M, N)) < 0.3] = 0.0
        G[:, N // 2:] *= np.float32(2.0 ** -112)
        G[: M // 2, : N // 2] *= np.float32(2.0 ** -98)
    else:
        for v in (np.inf, -np.inf, np.inf, np.nan):
            G[rng.integers(M // 2), rng.integers(N // 2)] = v
    tG = torch.from_numpy(G).to(DEV)
    ws = torch.full((max(256, lb.lba_grad_workspace_bytes_fast(M, N, K)),), 0x5A, dtype=torch.uint8, device=DEV)
    finite = np.where(np.isfinite(G), G, 0.0)
    for ste, plane, est in ((lb.STE_IDENTITY, None, 0), (lb.STE_IMMEDIATE_OF, of, 1), (lb.STE_COEF_PLANE, coef, 2)):
        c = gref.coefficients(A, B, ref.QFmt(*qp), ref.QFmt(*qa), est)
        tab = gref.decode_table()
        gc = np.where(c, G.astype(np.float64)[:, :, None], 0.0)
        with np.errstate(invalid="ignore"):
            wX, wW = (gc * tab[B][None]).sum(1), (gc * tab[A][:, None]).sum(0)
        aX, aW = gref.grad_abs(finite, A, B, ref.QFmt(*qp), ref.QFmt(*qa), est, c=c)
        for w in (ws, ws[:max(256, lb.lba_grad_workspace_bytes(M, N, K))], None):
            dX, dW = lb.grad(tG, tA, tB, ste, of_plane=plane, workspace=w)
            torch.cuda.synchronize()
            for got, want, scale, terms in ((dX.cpu().numpy(), wX, aX, N), (dW.cpu().numpy(), wW, aW, M)):
                ok = np.isfinite(want)
                assert ok.all() == (what != "infinite")
                assert np.array_equal(got[~ok], want[~ok].astype(np.float32), equal_nan=True), (ste, w is None)
                assert (np.abs(got[ok] - want[ok]) <= 2 * (terms + 1) * 2.0 ** -24 * scale[ok] + terms * 2.0 ** -126).all(), (ste, w is None)

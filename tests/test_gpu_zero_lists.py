"""Forward calls on packed FP16 carriers whose A holds zero codes: the steps a tile leaves out (lists of non-zero codes) against the
oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2401_14110_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ref():
    from oracle import lba_ref
    lba_ref.build()
    return lba_ref


def codes(rng, shape, zeros=0.0):
    """Random finite E4M3 codes of both signs; a share of them +0 and -0."""
    c = rng.integers(0, 256, shape, dtype=np.uint8)
    c = np.where((c & 0x7F) == 0x7F, c - 1, c).astype(np.uint8)
    z = rng.random(shape) < zeros
    return np.where(z, np.where(rng.random(shape) < 0.1, 0x80, 0), c).astype(np.uint8)


def check(ref, A, B, qp, qa, order=0):
    got = binding.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa, order=order)
    torch.cuda.synchronize()
    want = ref.gemm(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order)
    assert np.array_equal(got.cpu().numpy().view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


# quantizers that never saturate here, that do so at every step, and whose R_OF asks for the bound that follows the data
FORMATS = [((5, 7, 4, 0), (4, 7, -4, 0)), ((5, 7, 12, 0), (4, 1, 16, 0)), ((5, 7, 4, 0), (4, 7, 0, 0))]


# 64 x 64 tiles (two row sets), 32 x 64 (one), 48 x 64 (a set and a half) behind 64 x 64, 32 x 32 and 32 x 16; K at the edges
# of the 64-step tile, of its halves and of 16-byte rows
@pytest.mark.parametrize("M,N", [(4160, 512), (1000, 333), (3136, 512), (300, 200), (40, 70)])
@pytest.mark.parametrize("K", [64, 83, 96, 144, 272])
@pytest.mark.parametrize("qp,qa", FORMATS)
def test_shares_of_zeros(ref, M, N, K, qp, qa):
    rng = np.random.default_rng(M + K)
    A, B = codes(rng, (M, K)), codes(rng, (N, K), 0.05)
    # every share in one call: by rows, so that waves with and without lists stand side by side
    share = rng.choice([0.0, 0.2, 0.45, 0.5, 0.6, 0.9, 1.0], (-(-M // 32), 1)).repeat(32, 0)[:M]
    A = np.where(rng.random((M, K)) < share, 0, A).astype(np.uint8)
    if M * N > 100000:
        rows = np.sort(rng.choice(M, 96, replace=False))
        got = binding.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa).cpu().numpy()[rows]
        want = ref.gemm(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa))
        assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))
    else:
        check(ref, A, B, qp, qa)


# lists of every length, the full 64 and none among them, alone in a row set and next to others; zeros by columns, so that tiles
# with and without lists alternate along K (the sequential order; the chunked one has no lists and runs the same codes unrolled)
@pytest.mark.parametrize("order", [0, 1])
def test_list_lengths(ref, order):
    rng = np.random.default_rng(5)
    M, N, K = 1024, 1024, 320
    A, B = codes(rng, (M, K)), codes(rng, (N, K))
    A[A == 0] = 1
    for m in range(M):
        for t in range(K // 64):
            n = (m // 8 + 3 * t) % 65 if m % 8 == t else rng.integers(0, 40)
            A[m, 64 * t + rng.permutation(64)[n:]] = 0
    A[:, 128:192] = np.where(A[:, 128:192] == 0, 3, A[:, 128:192])
    rows = np.sort(rng.choice(M, 200, replace=False))
    got = binding.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), *FORMATS[0], order=order).cpu().numpy()[rows]
    want = ref.gemm(np.ascontiguousarray(A[rows]), B, ref.QFmt(*FORMATS[0][0]), ref.QFmt(*FORMATS[0][1]), order=order)
    assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


# chains that drift towards R_OF at different paces (columns of one sign and of both) behind half of zeros: lists the fixed bound covers, tiles
# left unrolled because it covers one part only, clamped lists, and the bound that follows the data (R_OF by the last format's bias)
@pytest.mark.parametrize("M,N", [(4160, 512), (3136, 512), (1000, 333)])
@pytest.mark.parametrize("ba", [-6, -5, -4, -3, -2, 0])
def test_lists_near_the_bound(ref, M, N, ba):
    rng = np.random.default_rng(M + ba + 10)
    K = 1100
    A = ((rng.integers(9, 15, (M, K)) << 3) | rng.integers(0, 8, (M, K))).astype(np.uint8)
    A = np.where(rng.random((M, K)) < rng.choice([0.5, 0.55, 0.8], (M, 1)), 0, A).astype(np.uint8)
    B = ((rng.integers(7, 13, (N, K)) << 3) | rng.integers(0, 8, (N, K))).astype(np.uint8)
    B = np.where(rng.random((N, K)) < rng.choice([0.0, 0.4, 0.5, 0.5], (N, 1)), B | 0x80, B).astype(np.uint8)
    rows = np.sort(rng.choice(M, 64, replace=False))
    qp, qa = (5, 7, 4, 0), (4, 7, ba, 0)
    got = binding.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa).cpu().numpy()[rows]
    want = ref.gemm(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa))
    assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


# im2col rows: zeros of the image, and whole taps outside it under a wide padding
@pytest.mark.parametrize("c,pad", [(16, 1), (48, 4), (20, 2)])
def test_convolutions(ref, c, pad):
    rng = np.random.default_rng(c)
    X, W = codes(rng, (6, 33, 31, c), 0.5), codes(rng, (136, 3, 3, c))
    qp, qa = FORMATS[0]
    got = binding.conv2d(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), qp, qa, stride=1, pad=pad)
    torch.cuda.synchronize()
    rows = ref.im2col_nhwc(X, 3, 3, 1, pad)
    pick = np.sort(rng.choice(rows.shape[0], 300, replace=False))
    want = ref.gemm(np.ascontiguousarray(rows[pick]), W.reshape(136, -1), ref.QFmt(*qp), ref.QFmt(*qa))
    assert np.array_equal(got.cpu().numpy().reshape(rows.shape[0], 136)[pick].view(np.uint32), np.ascontiguousarray(want).view(np.uint32))

"""Forward calls whose accumulator reaches beyond FP16's range (E >= 5) on packed FP16 carriers: chains that stay inside it, leave it in any
part of any tile, saturate or come back, against the oracle, bit for bit."""
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


def codes(rng, shape, lo, hi, signs=True, zeros=0.0):
    """E4M3 codes with exponent fields lo .. hi."""
    c = (rng.integers(lo, hi + 1, shape) << 3) | rng.integers(0, 7, shape)
    if signs:
        c = c | (rng.integers(0, 2, shape) << 7)
    return np.where(rng.random(shape) < zeros, 0, c).astype(np.uint8)


def compare(ref, A, B, qp, qa, order, rows=None):
    got = binding.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa, order=order)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    if rows is not None:
        got, A = got[rows], np.ascontiguousarray(A[rows])
    want = ref.gemm(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order)
    assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


# tiles of every kind: 64 x 64, 64 x 64 with 48 x 64 and 32 x 32 behind, 32 x 64, 32 x 32, 32 x 16; M = 10 has no mask
@pytest.mark.parametrize("M,N,kernel", [(4160, 512, "lba_wide_"), (12544, 256, "lba_wide_mixed_kernel"), (1000, 1024, "lba_wide_"), (300, 500, "lba_wide_"), (40, 70, "lba_wide_")])
@pytest.mark.parametrize("e,m", [(5, 10), (5, 7), (6, 3), (7, 10)])
def test_chains_around_the_range(ref, M, N, kernel, e, m):
    rng = np.random.default_rng(100 * e + m + M)
    K = 416 if M * N < 100000 else 352
    qp, qa = (6, 7, 10, 0), (e, m, 6, 0)
    assert binding.lba_plan_kernel_name(M, N, K, qp, qa, 0).startswith(kernel)
    # groups of rows: quiet; zeros by half; all products of one sign, which leave the range at a step that differs by group (E = 5
    # saturates in the end); up and down again
    A = codes(rng, (M, K), 4, 9)
    kind = (np.arange(M) // 16) % 5
    A = np.where((kind == 1)[:, None], codes(rng, (M, K), 4, 9, zeros=0.6), A)
    up = codes(rng, (M, K), 13, 15, signs=False)
    start = rng.integers(0, K // 2, -(-M // 16)).repeat(16)[:M]
    A = np.where(((kind == 2)[:, None]) & (np.arange(K) >= start[:, None]), up, A)
    A = np.where(((kind == 3)[:, None]), np.where(rng.random((M, K)) < 0.5, 0, up), A)
    A = np.where(((kind == 4)[:, None]), np.where(np.arange(K) < K // 2, up, up | 0x80), A).astype(np.uint8)
    B = codes(rng, (N, K), 12, 15, signs=False, zeros=0.1)
    B[::3] = codes(rng, B[::3].shape, 3, 8)
    rows = None if M * N < 100000 else np.sort(rng.choice(M, 80, replace=False))
    for order in (0, 1):
        compare(ref, A, B, qp, qa, order, rows)


# chains that leave the range and come back several times, at steps that differ by row and fall anywhere in a k-tile; a share of zeros
# by group of rows, so that tiles are lists on one stretch or the other; E = 5 saturates in between
@pytest.mark.parametrize("M,N", [(4160, 512), (12544, 256), (1000, 1024), (300, 500), (40, 70)])
@pytest.mark.parametrize("e,m", [(5, 10), (6, 7)])
def test_leaving_and_coming_back(ref, M, N, e, m):
    rng = np.random.default_rng(M + e)
    K = 787
    qp, qa = (6, 7, 10, 0), (e, m, 6, 0)
    A = codes(rng, (M, K), 12, 15, signs=False)
    period = rng.integers(40, 400, -(-M // 8)).repeat(8)[:M, None]          # a wave's groups of 8 rows differ
    down = (np.arange(K)[None, :] + rng.integers(0, 400, (M, 1))) % (2 * period) >= period
    A = np.where(down, A | 0x80, A)
    share = rng.choice([0.0, 0.5, 0.6, 0.9], (-(-M // 16), 1)).repeat(16, 0)[:M]
    A = np.where(rng.random((M, K)) < share, 0, A).astype(np.uint8)
    B = codes(rng, (N, K), 13, 15, signs=False)
    B[1::7] = codes(rng, B[1::7].shape, 2, 8)
    rows = None if M * N < 100000 else np.sort(rng.choice(M, 96, replace=False))
    for order in (0, 1):
        compare(ref, A, B, qp, qa, order, rows)


# both sides of the admission line (64 of the largest products inside the range) and ragged K
@pytest.mark.parametrize("K", [1, 31, 33, 64, 65, 147])
def test_admission_line_and_k(ref, K):
    rng = np.random.default_rng(K)
    A, B = codes(rng, (70, K), 0, 15, zeros=0.3), codes(rng, (50, K), 0, 15)
    names = set()
    for ba in (-3, 2, 6, 7, 9, 12):
        qp, qa = (6, 7, 9, 0), (5, 10, ba, 0)
        names.add((ba <= 6, binding.lba_plan_kernel_name(70, 50, K, qp, qa, 0).startswith("lba_wide_")))
        compare(ref, A, B, qp, qa, 0)
    if K >= 16:
        assert (False, True) not in names and (True, True) in names


@pytest.mark.parametrize("c", [16, 24])
def test_convolutions(ref, c):
    rng = np.random.default_rng(c)
    X, W = codes(rng, (5, 20, 19, c), 8, 15, signs=False, zeros=0.5), codes(rng, (72, 3, 3, c), 8, 15)
    qp, qa = (6, 7, 10, 0), (5, 10, 6, 0)
    got = binding.conv2d(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), qp, qa, stride=1, pad=1)
    torch.cuda.synchronize()
    want = ref.gemm(ref.im2col_nhwc(X, 3, 3, 1, 1), W.reshape(72, -1), ref.QFmt(*qp), ref.QFmt(*qa))
    assert np.array_equal(got.cpu().numpy().reshape(want.shape).view(np.uint32), np.ascontiguousarray(want).view(np.uint32))

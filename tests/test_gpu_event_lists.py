"""The recompute call for the overflow plane alone on codes with many zeros: tiles that leave steps of zero codes out beside tiles whose sums saturate,
where a step of a zero code is an overflow like any other, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2401_14110_amd import binding

pytestmark = pytest.mark.gpu

QP, QA = (5, 7, 4, 0), (4, 7, -2, 0)           # R_OF = 2^17 (2 - 2^-7), which a burst reaches and small codes do not


@pytest.fixture(scope="module")
def ref():
    from oracle import lba_ref
    lba_ref.build()
    return lba_ref


def same(got, want):
    return np.array_equal(np.ascontiguousarray(got).view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


def phases(rng, M, K):
    """A: small codes of both signs, then a burst of large ones of one sign that saturates the sums, then mostly zeros, then a burst of the
    other sign that brings the sums back; where each begins differs by row.  Half to nine tenths of the codes outside the bursts are zero."""
    small = ((rng.integers(3, 8, (M, K)) << 3) | rng.integers(0, 8, (M, K)) | (rng.integers(0, 2, (M, K)) << 7)).astype(np.uint8)
    large = ((rng.integers(14, 16, (M, K)) << 3) | rng.integers(0, 7, (M, K))).astype(np.uint8)
    A = np.where(rng.random((M, K)) < rng.choice([0.5, 0.6, 0.9], (M, 1)), 0, small)
    start = rng.integers(0, max(1, K - 100), (M, 1)) // rng.choice([1, 16, 64], (M, 1)) * rng.choice([1, 16, 64], (M, 1))
    k = np.arange(K)[None, :] - start
    A = np.where((k >= 0) & (k < 60), large, A)
    A = np.where((k >= 60) & (k < 220), np.where(rng.random((M, K)) < 0.9, 0, small), A)
    A = np.where((k >= 220) & (k < 250), large | 0x80, A)
    quiet = (np.arange(M) // 16) % 3 == 0                      # whole waves without a burst
    return np.where(quiet[:, None], np.where(rng.random((M, K)) < 0.6, 0, small), A).astype(np.uint8)


def weights(rng, N, K):
    return ((rng.integers(9, 14, (N, K)) << 3) | rng.integers(0, 8, (N, K))).astype(np.uint8)


def some(rng, M):
    return np.array(sorted({0, M // 2, M - 40, M - 1} | set(int(r) for r in rng.integers(0, M, 60))))


# 64 x 64 workgroups, and those with 32 x 32 behind them; 16-byte rows and not; K of one tile and of many
@pytest.mark.parametrize("M,N,kernel", [(20000, 60, "lba_half_bwd_kernel"), (17000, 72, "lba_half_bwd_mixed_kernel"), (27000, 64, "lba_half_bwd_mixed_kernel")])
@pytest.mark.parametrize("K", [64, 400, 403, 640])
def test_rows(ref, M, N, kernel, K):
    rng = np.random.default_rng([M, K])
    A, B = phases(rng, M, K), weights(rng, N, K)
    assert binding.lba_plan_kernel_name(M, N, K, QP, QA, 0, 3).startswith(kernel)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = some(rng, M)
    C, of, _, ws = binding.gemm_bwd_ws(dA, dB, QP, QA, want_uf=False)
    torch.cuda.synchronize()
    want = ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*QP), ref.QFmt(*QA))
    assert same(C.cpu().numpy()[rows], want[0]) and same(of.cpu().numpy()[:, rows], want[1])
    zero = np.zeros((-(-K // 32) * 32, len(rows)), dtype=bool)
    zero[:K] = (A[rows] == 0).T
    bits = (want[1][:, None] >> np.arange(32, dtype=np.uint32)[None, :, None, None]) & 1
    if K > 64:                                                 # events at steps of zero codes, which a list would not have
        assert (bits.reshape(-1, len(rows), N)[zero] != 0).any() and (want[1] == 0).any()
    # the maps of dirty bricks that the call leaves behind: the gradient products that rely on them equal those of the plane itself
    G = torch.from_numpy(rng.standard_normal((M, N)).astype(np.float32)).cuda()
    for x, y in zip(binding.grad_premapped(G, dA, dB, of, ws), binding.grad(G, dA, dB, binding.STE_IMMEDIATE_OF, of_plane=of)):
        x, y = x.double(), y.double()
        assert float((x - y).norm() / y.norm()) < 1e-5         # 32-bit sums of at most 27000 terms in another order


@pytest.mark.parametrize("c", [16, 20])
def test_tensors(ref, c):
    rng = np.random.default_rng(c)
    n, h, w, cout = 6, 53, 55, 72
    X = phases(rng, n * h * w, c).reshape(n, h, w, c)
    X = np.where(rng.random((n, h, w, 1)) < 0.05, 0x77, X).astype(np.uint8)
    W = weights(rng, cout, 9 * c).reshape(cout, 3, 3, c)
    d = binding.lba_conv2d_desc(n, h, w, c, 3, 3, 1, 1)
    M, K = n * h * w, 9 * c
    dX, dW = torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda()
    Y = torch.empty(M, cout, dtype=torch.float32, device="cuda")
    of = torch.full((-(-K // 32), M, cout), -1, dtype=torch.int32, device="cuda")
    rc = binding.lib().lba_conv2d_bwd(dX.data_ptr(), dW.data_ptr(), Y.data_ptr(), of.data_ptr(), None, d, cout, binding.qfmt(QP), binding.qfmt(QA), 0, None)
    torch.cuda.synchronize()
    assert rc == binding.OK
    rows = some(rng, M)
    want = ref.gemm_bwd(np.ascontiguousarray(ref.im2col_nhwc(X, 3, 3, 1, 1)[rows]), W.reshape(cout, -1), ref.QFmt(*QP), ref.QFmt(*QA))
    assert same(Y.cpu().numpy()[rows], want[0]) and same(of.cpu().numpy()[:, rows], want[1])
    assert (want[1] != 0).any() and (want[1] == 0).any()

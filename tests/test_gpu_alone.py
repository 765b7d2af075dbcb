"""Launches on packed FP16 carriers whose large workgroups number at most one per CU (csrc/lba_half_alone.hip) against the oracle, bit for bit, on both
sides of the rule that chooses them."""
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


def codes(rng, shape, zeros):
    """Random finite E4M3 codes of both signs, a share of them zero."""
    c = rng.integers(0, 256, shape, dtype=np.uint8)
    c = np.where((c & 0x7F) == 0x7F, c - 1, c)
    return np.where(rng.random(shape) < zeros, 0, c).astype(np.uint8)


def same(got, want):
    return np.array_equal(np.ascontiguousarray(got).view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


def some(rng, M):
    return np.array(sorted({0, 1, min(63, M - 1), M // 2, M - 2, M - 1} | set(int(r) for r in rng.integers(0, M, 40))))


# never, now and then and nearly always saturated; the last one's R_OF asks for the bound that follows the data
FORMATS = [((5, 7, 4, 0), (4, 7, -4, 0)), ((5, 7, 12, 0), (4, 1, 16, 0)), ((5, 7, 4, 0), (4, 7, 0, 0))]


# 1 to 256 and 257 workgroups of 64 x 64; K at the edges of a k-tile and of its halves, 16-byte rows and not
@pytest.mark.parametrize("M,N,alone", [(33, 18, True), (70, 130, True), (16384, 64, True), (4096, 250, True), (16400, 64, False)])
@pytest.mark.parametrize("K", [16, 33, 64, 83, 144, 272])
@pytest.mark.parametrize("zeros", [0.1, 0.6])
def test_recompute(ref, M, N, alone, K, zeros):
    rng = np.random.default_rng([M, K])
    A, B = codes(rng, (M, K), zeros), codes(rng, (N, K), 0.1)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = some(rng, M)
    for qp, qa in FORMATS:
        for order in (0, 1):
            for events in (1, 3):
                assert ("alone" in binding.lba_plan_kernel_name(M, N, K, qp, qa, order, events)) == alone
        want = ref.gemm_bwd(A[rows], B, ref.QFmt(*qp), ref.QFmt(*qa))
        for uf in (True, False):
            got = binding.gemm_bwd(dA, dB, qp, qa, want_uf=uf)
            torch.cuda.synchronize()
            assert same(got[0].cpu().numpy()[rows], want[0]), (qp, qa, uf)
            for i in range(1, 3 if uf else 2):
                assert same(got[i].cpu().numpy()[:, rows], want[i]), (qp, qa, uf, i)
        want = ref.gemm_bwd(A[rows], B, ref.QFmt(*qp), ref.QFmt(*qa), order=1, level2=True)
        for uf in (True, False):
            got = binding.gemm_bwd_chunked(dA, dB, qp, qa, want_uf=uf)
            torch.cuda.synchronize()
            assert same(got[0].cpu().numpy()[rows], want[0]), (qp, qa, uf)
            for i in range(1, 5):
                if got[i] is not None:
                    assert same(got[i].cpu().numpy()[:, rows], want[i]), (qp, qa, uf, i)


# products that Q_prod truncates: forward on 64 x 64 workgroups (a batch counts all of its own; the fewest have waves that stage), and recompute
@pytest.mark.parametrize("batch,M,N,alone", [(1, 100, 70, False), (1, 401, 450, True), (1, 16384, 64, True), (1, 16385, 64, False), (4, 256, 1024, True), (5, 256, 1024, False)])
@pytest.mark.parametrize("K", [48, 83, 160])
def test_truncated_products(ref, batch, M, N, alone, K):
    rng = np.random.default_rng([batch, M, K])
    A, B = codes(rng, (batch, M, K), 0.5), codes(rng, (batch, N, K), 0.1)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = some(rng, M)
    for qp, qa in [((5, 4, 4, 0), (4, 7, -4, 0)), ((5, 4, 4, 0), (4, 7, 0, 0))]:
        if batch == 1:
            assert ("alone" in binding.lba_plan_kernel_name(M, N, K, qp, qa, 0)) == (alone or (M == 100 and K <= 64))
        for order in (0, 1):
            got = binding.gemm_batched(dA, dB, qp, qa, order=order).cpu().numpy()
            for b in range(batch):
                assert same(got[b][rows], ref.gemm(A[b][rows], B[b], ref.QFmt(*qp), ref.QFmt(*qa), order=order)), (qa, order, b)
        if batch == 1:
            got = binding.gemm_bwd(dA[0], dB[0], qp, qa)
            torch.cuda.synchronize()
            want = ref.gemm_bwd(A[0][rows], B[0], ref.QFmt(*qp), ref.QFmt(*qa))
            assert same(got[0].cpu().numpy()[rows], want[0])
            assert same(got[1].cpu().numpy()[:, rows], want[1]) and same(got[2].cpu().numpy()[:, rows], want[2])


# one workgroup of 48 x 64 per CU and fewer than 256 of 32 x 32 behind them, and as many
@pytest.mark.parametrize("M,N,alone", [(18050, 24, True), (18920, 32, True), (20448, 17, True), (20449, 24, False), (18050, 40, False)])
@pytest.mark.parametrize("K", [64, 83, 208])
def test_one_workgroup_of_48_rows_per_cu(ref, M, N, alone, K):
    rng = np.random.default_rng([M, N, K])
    A, B = codes(rng, (M, K), 0.5), codes(rng, (N, K), 0.1)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = np.array(sorted(set(some(rng, M)) | {12287, 12288, 12289}))
    for qp, qa in FORMATS:
        for order in (0, 1):
            assert ("alone" in binding.lba_plan_kernel_name(M, N, K, qp, qa, order)) == alone
            got = binding.gemm(dA, dB, qp, qa, order=order).cpu().numpy()[rows]
            assert same(got, ref.gemm(A[rows], B, ref.QFmt(*qp), ref.QFmt(*qa), order=order)), (qa, order)


# the same from a tensor: whole taps and filter rows that pieces span, forward and recompute
@pytest.mark.parametrize("n,h,w,c,cout", [(3, 80, 79, 16, 24), (3, 80, 79, 6, 24), (1, 20, 21, 16, 70), (2, 20, 21, 6, 70)])
def test_convolutions(ref, n, h, w, c, cout):
    rng = np.random.default_rng([h, c])
    X, W = codes(rng, (n, h, w, c), 0.5), codes(rng, (cout, 3, 3, c), 0.1)
    dX, dW = torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda()
    A = ref.im2col_nhwc(X, 3, 3, 1, 1)
    rows = some(rng, A.shape[0])
    A, B = np.ascontiguousarray(A[rows]), W.reshape(cout, -1)
    for qp, qa in FORMATS:
        for order in (0, 1):
            got = binding.conv2d(dX, dW, qp, qa, stride=1, pad=1, order=order)
            assert same(got.cpu().numpy().reshape(-1, cout)[rows], ref.gemm(A, B, ref.QFmt(*qp), ref.QFmt(*qa), order=order)), (qa, order)
        want = ref.gemm_bwd(A, B, ref.QFmt(*qp), ref.QFmt(*qa))
        got = binding.conv2d(dX, dW, qp, qa, stride=1, pad=1, planes=True)
        torch.cuda.synchronize()
        assert same(got[0].cpu().numpy().reshape(-1, cout)[rows], want[0]), qa
        for i in (1, 2):
            assert same(got[i].cpu().numpy().reshape(-1, n * h * w, cout)[:, rows], want[i]), (qa, i)

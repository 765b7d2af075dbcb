"""The smallest forward grids under nearest-even (waves of their own stage) against the oracle, bit for bit."""
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


# M = 7 (rounded by the bfloat16 conversion) and M = 9, products flushed or not; accumulators never, now and then and nearly always saturated
FORMATS = [((5, 7, 4, 1), (4, 7, -4, 1)), ((5, 7, 12, 1), (5, 9, 12, 1)), ((5, 7, 12, 1), (4, 7, 2, 1)), ((6, 7, 24, 1), (5, 9, 19, 1)), ((6, 7, 40, 1), (4, 7, -4, 1))]


# one tile, 32 x 16 tiles with ragged edges, 32 x 32 tiles; K at the edges of a k-tile, of its halves, of four tiles ahead
@pytest.mark.parametrize("M,N,cols", [(64, 64, 2), (1, 16, 2), (40, 70, 2), (300, 201, 2), (512, 482, 4), (520, 451, 4)])
@pytest.mark.parametrize("K", [16, 33, 64, 83, 272, 331])
def test_small_grids(ref, M, N, cols, K):
    rng = np.random.default_rng(1000 * M + K)
    A, B = (rng.integers(0, 256, s, dtype=np.uint8) for s in ((M, K), (N, K)))
    A = np.where(rng.random(A.shape) < 0.3, 0, A).astype(np.uint8)
    rows = np.sort(rng.choice(M, min(M, 64), replace=False))
    for qp, qa in FORMATS:
        assert binding.lba_plan_kernel_name(M, N, K, qp, qa, 0).startswith("lba_fast_staged_kernel<%d" % cols)
        got = binding.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa).cpu().numpy()[rows]
        want = ref.gemm(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa))
        assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


def test_batch_off_alignment(ref):
    rng = np.random.default_rng(7)
    nb, M, N, K = 3, 70, 50, 75
    buf = rng.integers(0, 256, 2 * nb * (M + N) * K + 1, dtype=np.uint8)
    dev = torch.from_numpy(buf).cuda()
    A, B = buf[1:1 + nb * M * K].reshape(nb, M, K), buf[1 + nb * M * K:1 + nb * (M + N) * K].reshape(nb, N, K)
    dA, dB = dev[1:1 + nb * M * K].view(nb, M, K), dev[1 + nb * M * K:1 + nb * (M + N) * K].view(nb, N, K)
    qp, qa = FORMATS[2]
    got = binding.gemm_batched(dA, dB, qp, qa).cpu().numpy()
    for b in range(nb):
        want = ref.gemm(np.ascontiguousarray(A[b]), np.ascontiguousarray(B[b]), ref.QFmt(*qp), ref.QFmt(*qa))
        assert np.array_equal(got[b].view(np.uint32), np.ascontiguousarray(want).view(np.uint32))

"""The overflow planes of the chunked order alone, on plain grids and on grids with a tail of 32 x 32 tiles, bit for bit."""
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


# 512 workgroups of 64 x 64 and the next, one tail tile and several, rows and columns off the tiles; the last two: a tail would have more than one to a CU
@pytest.mark.parametrize("M,N,tail", [(64 * 512, 64, False), (64 * 512 + 1, 64, True), (64 * 530 + 45, 60, True), (64 * 260 + 9, 130, True), (64 * 570, 64, True), (64 * 600, 64, False),
                                      (12 * 64 + 40, 64 * 52, False)])
@pytest.mark.parametrize("K", [16, 63, 100, 288])
def test_overflow_planes(ref, M, N, tail, K):
    rng = np.random.default_rng([M, N, K])
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 72, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = np.unique(np.concatenate([[0, M - 1, M - 40, 64 * 512 - 1 if M > 64 * 512 else 1], rng.choice(M, 24)]))
    for bias in (5, 9, 12):                                    # few overflows, some, most sums saturate
        qp, qa = (5, 7, 12, 0), (4, 7, bias, 0)
        assert (binding.lba_plan_query(M, N, K, qp, qa, 1, 3)["tail_blocks"] > 0) == tail
        c, of, uf, of2, uf2 = binding.gemm_bwd_chunked(dA, dB, qp, qa, want_uf=False)
        torch.cuda.synchronize()
        want = ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa), order=1, level2=True)
        assert uf is None and uf2 is None
        assert np.array_equal(c.cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(want[0]).view(np.uint32))
        assert np.array_equal(of.cpu().numpy()[:, rows].view(np.uint32), want[1]) and np.array_equal(of2.cpu().numpy()[:, rows].view(np.uint32), want[3])


# a format that packed carriers hold without an underflow plane only: both levels of the overflow planes, on few workgroups, a plain grid and one with a tail
@pytest.mark.parametrize("M,N", [(33, 37), (64 * 200 + 1, 60), (64 * 300, 64), (64 * 530 + 45, 60)])
@pytest.mark.parametrize("K", [15, 100, 1050])
def test_products_far_below_the_sums(ref, M, N, K):
    if K > 1000 and M > 64 * 200 + 1:
        K = 550                                                # (more than 32 chunks: a second word of the second level, on the smaller ones)
    rng = np.random.default_rng([M, N, K])
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 110, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    A[::3] = rng.integers(124, 127, A[::3].shape)             # rows whose sums reach R_OF on the longest chains, at the second level
    B[::2] = rng.integers(124, 127, B[::2].shape)
    qp, qa = (5, 7, 1, 0), (4, 7, -10, 0)
    assert "half" in binding.lba_plan_kernel_name(M, N, K, qp, qa, 1, 3) and "half" not in binding.lba_plan_kernel_name(M, N, K, qp, qa, 1, 1)
    rows = np.unique(np.concatenate([[0, M - 1], rng.choice(M, min(M, 30), replace=False)]))
    c, of, _, of2, _ = binding.gemm_bwd_chunked(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa, want_uf=False)
    want = ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa), order=1, level2=True)
    assert np.array_equal(c.cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(want[0]).view(np.uint32))
    assert np.array_equal(of.cpu().numpy()[:, rows].view(np.uint32), want[1]) and np.array_equal(of2.cpu().numpy()[:, rows].view(np.uint32), want[3])
    assert want[3].any() == (K > 500)

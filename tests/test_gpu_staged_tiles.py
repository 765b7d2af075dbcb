"""Forward grids whose k-tiles other waves stage: chains over many tiles and their stages, with and without the clamp, bit for bit."""
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


# R_OF far above the sums (no clamp), near them (the bounds hold in some tiles and not in others), and saturated most of the time
@pytest.mark.parametrize("bias", [-2, 5, 7, 9, 12])
@pytest.mark.parametrize("rnd", [0, 1])
@pytest.mark.parametrize("M,N", [(33, 20), (288, 160), (500, 450)])
@pytest.mark.parametrize("K", [1, 64, 65, 129, 256, 321, 577, 1100])
def test_tiles(ref, M, N, K, rnd, bias):
    rng = np.random.default_rng(K + M)
    # codes of values up to 2 (growing along the chain, so that the bounds are passed inside it)
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 64, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    qp, qa = (5, 7, 12, rnd), (4, 7, bias, rnd)
    kernel = "lba_half_staged_kernel" if rnd == 0 else "lba_fast_staged_kernel"
    assert binding.lba_plan_kernel_name(M, N, K, qp, qa, 0).startswith(kernel)
    rows = np.sort(rng.choice(M, min(M, 40), replace=False))
    got = binding.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa).cpu().numpy()[rows]
    want = ref.gemm(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa))
    assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


# the chunked order, and products that Q_prod truncates: (the inputs' format, Q_prod's mantissa bits), 4: E4M3
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("M,N,K", [(33, 20, 15), (120, 100, 97), (350, 350, 321), (64, 64, 513), (500, 400, 577), (700, 600, 65)])
@pytest.mark.parametrize("ea,qpm", [(4, 4), (3, 5), (3, 7), (4, 7)])
@pytest.mark.parametrize("bias", [5, 9, 12])
def test_orders_and_truncated_products(ref, ea, qpm, bias, M, N, K, order):
    rng = np.random.default_rng(K + M + ea)
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 64 if ea == 4 else 80, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    # (a range of Q_prod that packed carriers hold with either format of the operands)
    qp, qa, fmt = (5, qpm, 12 if ea == 4 else 6, 0), (4, 7, bias, 0), (ea, 7 - ea, 8 if ea == 4 else 4)
    name = binding.lba_plan_kernel_name_in(M, N, K, fmt, fmt, qp, qa, order)
    if K == 65 and (ea, qpm) == (4, 7):
        assert name.startswith("lba_half_staged_kernel<4,") and name.endswith(", %d>" % order)
    if K >= 224 and ((ea, qpm, order) != (4, 7, 1) or M > 64):   # (few outputs in chunks: lba_kpar_kernel)
        assert name.startswith("lba_half_staged_kernel<2,") and name.endswith(", %d>" % order)
    rows = np.sort(rng.choice(M, min(M, 40), replace=False))
    got = binding.gemm_in(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), fmt, fmt, qp, qa, order=order).cpu().numpy()[rows]
    want = ref.gemm_in(np.ascontiguousarray(A[rows]), B, ref.InFmt(*fmt), ref.InFmt(*fmt), ref.QFmt(*qp), ref.QFmt(*qa), order=order)
    assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


# chunks of im2col rows (whole taps, pieces that span filter rows) and of a batch, whose tiles are 32 x 32
@pytest.mark.parametrize("bias", [5, 9, 12])
@pytest.mark.parametrize("n,h,w,c,cout,k", [(1, 9, 7, 32, 40, 3), (2, 14, 15, 24, 100, 3), (3, 20, 17, 64, 128, 3), (1, 30, 31, 6, 64, 7)])
def test_chunks_conv(ref, n, h, w, c, cout, k, bias):
    rng = np.random.default_rng(c + cout)
    X, W = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 64, s)).astype(np.uint8) for s in ((n, h, w, c), (cout, k, k, c)))
    qp, qa = (5, 7, 12, 0), (4, 7, bias, 0)
    got = binding.conv2d(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), qp, qa, stride=1, pad=k // 2, order=1).cpu().numpy()
    want = ref.gemm(ref.im2col_nhwc(X, k, k, 1, k // 2), W.reshape(cout, -1), ref.QFmt(*qp), ref.QFmt(*qa), order=1)
    assert np.array_equal(got.reshape(-1, cout).view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


@pytest.mark.parametrize("bias", [5, 9, 12])
@pytest.mark.parametrize("batch,M,N,K", [(3, 40, 70, 16), (5, 64, 64, 97), (20, 100, 64, 200)])
def test_chunks_batched(ref, batch, M, N, K, bias):
    rng = np.random.default_rng(K)
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 64, s)).astype(np.uint8) for s in ((batch, M, K), (batch, N, K)))
    qp, qa = (5, 7, 12, 0), (4, 7, bias, 0)
    got = binding.gemm_batched(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), qp, qa, order=1).cpu().numpy()
    for i in range(batch):
        want = ref.gemm(A[i], B[i], ref.QFmt(*qp), ref.QFmt(*qa), order=1)
        assert np.array_equal(got[i].view(np.uint32), np.ascontiguousarray(want).view(np.uint32))

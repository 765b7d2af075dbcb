"""The overflow plane alone from the entry points for other operand formats and convolutions, in formats that packed carriers hold only without an
underflow plane among them, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2401_14110_amd import binding

pytestmark = pytest.mark.gpu
DEEP = ((5, 7, 1, 0), (4, 7, -10, 0))       # a product can fall far below the sum's smallest unit


@pytest.fixture(scope="module")
def ref():
    from oracle import lba_ref
    lba_ref.build()
    return lba_ref


# few workgroups of 64 x 64, 257 to 320, up to 512 and more
@pytest.mark.parametrize("M,N", [(33, 37), (64 * 200 + 1, 60), (64 * 300, 64), (64 * 400 + 9, 63), (64 * 560, 64)])
@pytest.mark.parametrize("fmt,qp,qa", [((4, 3, 7), *DEEP), ((4, 3, 7), (5, 7, 12, 0), (4, 7, 9, 0)), ((3, 4, 3), (5, 7, 1, 0), (4, 7, 2, 0)), ((3, 4, 3), (5, 7, 1, 0), (5, 10, 5, 0))])
def test_other_formats(ref, fmt, qp, qa, M, N):
    K = 77
    rng = np.random.default_rng([M, N])
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 100, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    if (qp, qa) == DEEP:
        assert "half" not in binding.lba_plan_kernel_name_in(M, N, K, fmt, fmt, qp, qa, 0, 1) and "half" in binding.lba_plan_kernel_name_in(M, N, K, fmt, fmt, qp, qa, 0, 3)
    c, of, uf = binding.gemm_in(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), fmt, fmt, qp, qa, planes=True, uf_plane=False)
    rows = np.unique(np.concatenate([[0, M - 1], rng.choice(M, min(M, 60), replace=False)]))
    want = ref.gemm_in(np.ascontiguousarray(A[rows]), B, ref.InFmt(*fmt), ref.InFmt(*fmt), ref.QFmt(*qp), ref.QFmt(*qa), planes=True)
    assert uf is None
    assert np.array_equal(c.cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(want[0]).view(np.uint32))
    assert np.array_equal(of.cpu().numpy()[:, rows].view(np.uint32), want[1])


@pytest.mark.parametrize("c", [16, 20, 3])
@pytest.mark.parametrize("n,h,w,cout", [(1, 7, 9, 20), (3, 64, 68, 64), (5, 64, 64, 60), (7, 64, 64, 64)])
@pytest.mark.parametrize("qp,qa", [DEEP, ((5, 7, 12, 0), (4, 7, 9, 0)), ((5, 4, 12, 0), (4, 7, 9, 0)), ((5, 7, 12, 0), (5, 10, 9, 0))])
def test_convolutions(ref, qp, qa, n, h, w, cout, c):
    rng = np.random.default_rng([n, c])
    X, W = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 100, s)).astype(np.uint8) for s in ((n, h, w, c), (cout, 3, 3, c)))
    tX, tW = torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda()
    M, K = n * h * w, 9 * c
    Y = torch.empty(M, cout, device="cuda")
    of = torch.empty((K + 31) // 32, M, cout, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert binding.lba_conv2d_bwd(tX.data_ptr(), tW.data_ptr(), Y.data_ptr(), of.data_ptr(), None, (n, h, w, c, 3, 3, 1, 1), cout, qp, qa, 0, stream) == 0
    A = ref.im2col_nhwc(X, 3, 3, 1, 1)
    rows = np.unique(np.concatenate([[0, M - 1], rng.choice(M, min(M, 60), replace=False)]))
    want = ref.gemm_bwd(np.ascontiguousarray(A[rows]), W.reshape(cout, -1), ref.QFmt(*qp), ref.QFmt(*qa))
    assert np.array_equal(Y.cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(want[0]).view(np.uint32))
    assert np.array_equal(of.cpu().numpy()[:, rows].view(np.uint32), want[1])

"""Both planes of matrices that end inside a lane's columns, on every grid of the packed recompute call, bit for bit; nothing beyond a plane is written."""
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


GUARD = 0x5A5AA5A5


def guarded(*shape):
    """A plane inside a larger buffer of guard words, and a check that the words around it are as they were."""
    n = int(np.prod(shape))
    buf = torch.full((n + 512,), GUARD, dtype=torch.int32, device="cuda")

    def untouched():
        return bool((buf[:256] == GUARD).all()) and bool((buf[256 + n:] == GUARD).all())

    return buf[256:256 + n].view(*shape), untouched


def ptr(t):
    return t.data_ptr()


# 32 x 32 workgroups alone, 64 x 64 ones, 64 x 64 ones before 32 x 32; matrices that end in the first tile, behind whole ones and one to three columns into a tile
@pytest.mark.parametrize("M", [35, 64 * 390, 64 * 520 + 3])
@pytest.mark.parametrize("N", [1, 3, 5, 33, 34, 35, 61, 62, 63, 66, 97, 126, 129])
def test_widths(ref, M, N):
    K = 70
    rng = np.random.default_rng([M, N, K])
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 72, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    wide = torch.zeros(-(-N // 64) * 64, K, dtype=torch.uint8, device="cuda")      # the same columns in a width of whole tiles
    wide[:N] = dB
    rows = np.unique(np.concatenate([[0, 1, M - 2, M - 1], rng.choice(M, 30, replace=False)]))
    qp, qa = (5, 7, 12, 0), (4, 7, 9, 0)
    stream = torch.cuda.current_stream().cuda_stream
    for order, right in [(0, ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa))),
                         (1, ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa), order=1, level2=True))]:
        assert binding.lba_plan_kernel_name(M, N, K, qp, qa, order, 1).startswith("lba_half_bwd_")
        c = torch.empty(M, N, device="cuda")
        planes = [guarded(w, M, N) for w in (3, 3, 1, 1)[:4 if order else 2]]
        at = [ptr(t) for t, _ in planes]
        if order:
            assert binding.lba_gemm_bwd_chunked(ptr(dA), ptr(dB), ptr(c), *at, M, N, K, qp, qa, stream) == binding.OK
        else:
            assert binding.lba_gemm_bwd(ptr(dA), ptr(dB), ptr(c), *at, M, N, K, qp, qa, 0, stream) == binding.OK
        other = binding.gemm_bwd_chunked(dA, wide, qp, qa) if order else binding.gemm_bwd(dA, wide, qp, qa)
        torch.cuda.synchronize()
        assert np.array_equal(c.cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(right[0]).view(np.uint32))
        assert torch.equal(c.view(torch.int32), other[0][:, :N].contiguous().view(torch.int32))
        for (g, untouched), r, o in zip(planes, right[1:], other[1:]):
            assert untouched()
            assert np.array_equal(g.cpu().numpy()[:, rows].view(np.uint32), r) and torch.equal(g, o[:, :, :N])


# chains of more than 512 steps: 32 x 32 workgroups on the smallest grids, 64 x 64 ones alone on their CUs and more of them
@pytest.mark.parametrize("M", [64 * 160, 64 * 200 + 3, 64 * 256, 64 * 300])
@pytest.mark.parametrize("N", [34, 61])
def test_deep_chains(ref, M, N):
    K = 515
    rng = np.random.default_rng([M, N, K])
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 72, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = np.unique(np.concatenate([[0, 1, M - 2, M - 1], rng.choice(M, 30, replace=False)]))
    qp, qa = (5, 7, 12, 0), (4, 7, 9, 0)
    for order in (0, 1):
        right = ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa), **({"order": 1, "level2": True} if order else {}))
        for uf in (True, False):
            got = binding.gemm_bwd_chunked(dA, dB, qp, qa, want_uf=uf) if order else binding.gemm_bwd(dA, dB, qp, qa, want_uf=uf)
            torch.cuda.synchronize()
            assert np.array_equal(got[0].cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(right[0]).view(np.uint32))
            for g, r in zip(got[1:], right[1:]):
                assert g is None or np.array_equal(g.cpu().numpy()[:, rows].view(np.uint32), r)

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

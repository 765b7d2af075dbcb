"""Recompute calls of few workgroups: 32 x 32 tiles (packed and FP32 carriers), and 64 x 64 ones for the overflow plane alone of more than 192, bit for bit; with the
brick maps that gradients read."""
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


# one tile and its edges, 191 to 256 workgroups of 64 x 64
@pytest.mark.parametrize("M,N", [(2, 4), (31, 32), (33, 36), (64 * 191 + 33, 28), (64 * 192 + 1, 60), (960, 64 * 16), (64 * 255 + 1, 64)])
@pytest.mark.parametrize("K", [15, 64, 97, 160])
def test_small_recompute(ref, M, N, K):
    rng = np.random.default_rng([M, N, K])
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 72, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = np.unique(np.concatenate([[0, M - 1, M // 2], rng.choice(M, min(M, 40), replace=False)]))
    blocks = ((M + 63) // 64) * ((N + 63) // 64)
    for bias in (5, 9, 12):                                    # few overflows, some, most sums saturate
        qp, qa = (5, 7, 12, 0), (4, 7, bias, 0)
        for order, events, tile in [(0, 1, 32), (0, 3, 32 if blocks <= 192 else 64), (1, 1, 32), (1, 3, 32)]:
            assert binding.lba_plan_query(M, N, K, qp, qa, order, events)["tile_m"] == tile
            assert binding.lba_plan_kernel_name(M, N, K, qp, qa, order, events).startswith("lba_half_bwd_alone_kernel<%d," % (tile // 16))
        want = ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa))
        chunks = ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa), order=1, level2=True)
        for uf in (True, False):
            for got, right in [(binding.gemm_bwd(dA, dB, qp, qa, want_uf=uf), want), (binding.gemm_bwd_ws(dA, dB, qp, qa, want_uf=uf)[:3], want),
                               (binding.gemm_bwd_chunked(dA, dB, qp, qa, want_uf=uf), chunks)]:
                torch.cuda.synchronize()
                assert np.array_equal(got[0].cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(right[0]).view(np.uint32))
                for g, r in zip(got[1:], right[1:]):
                    assert g is None or np.array_equal(g.cpu().numpy()[:, rows].view(np.uint32), r)
    # the maps: gradients through them are those of the plane alone
    _, of, _, ws = binding.gemm_bwd_ws(dA, dB, qp, qa, want_uf=False)
    G = torch.from_numpy(rng.integers(-4, 5, (M, N)).astype(np.float32)).cuda()   # (every product and sum is exact in FP32)
    for a, b in zip(binding.grad_premapped(G, dA, dB, of, ws), binding.grad(G, dA, dB, binding.STE_IMMEDIATE_OF, of_plane=of)):
        assert torch.equal(a, b)


# FP32 carriers (nearest-even, a wide accumulator) up to 320 and 512 workgroups of 64 x 64, both planes on packed carriers from 257 to 384
@pytest.mark.parametrize("qp,qa", [((5, 7, 12, 1), (4, 7, 9, 1)), ((5, 7, 12, 0), (5, 10, 9, 0)), ((5, 7, 12, 0), (4, 7, 9, 0))])
@pytest.mark.parametrize("M,N", [(2, 9), (31, 36), (65, 60), (64 * 256 + 1, 64), (64 * 320, 60), (64 * 320 + 1, 64), (64 * 384, 64), (64 * 511 + 1, 64)])
@pytest.mark.parametrize("K", [15, 64, 97])
def test_small_grids(ref, M, N, K, qp, qa):
    rng = np.random.default_rng([M, N, K])
    A, B = ((rng.integers(0, 2, s) * 128 + rng.integers(0, 72, s)).astype(np.uint8) for s in ((M, K), (N, K)))
    rows = np.unique(np.concatenate([[0, M - 1, M // 2], rng.choice(M, min(M, 40), replace=False)]))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    blocks, packed = ((M + 63) // 64) * ((N + 63) // 64), qp[3] == 0 and qa[0] == 4
    want = ref.gemm_bwd(np.ascontiguousarray(A[rows]), B, ref.QFmt(*qp), ref.QFmt(*qa))
    for events in (1, 3):
        small = 256 < blocks <= 384 and events == 1 if packed else blocks <= (512 if events == 1 else 320)
        plan = binding.lba_plan_query(M, N, K, qp, qa, 0, events)
        if small:                                              # 32 x 32 throughout
            assert plan["tail_blocks"] == ((M + 31) // 32) * ((N + 31) // 32) == plan["grid_x"]
        got = binding.gemm_bwd(dA, dB, qp, qa, want_uf=events == 1)
        torch.cuda.synchronize()
        assert np.array_equal(got[0].cpu().numpy()[rows].view(np.uint32), np.ascontiguousarray(want[0]).view(np.uint32))
        for g, r in zip(got[1:], want[1:]):
            assert g is None or np.array_equal(g.cpu().numpy()[:, rows].view(np.uint32), r)

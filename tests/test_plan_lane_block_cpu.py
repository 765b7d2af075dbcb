"""Which lane block plain grids of 513 to 1024 workgroups of 64 x 64 take: host logic only."""
import pytest

from paper_2401_14110_amd import binding

FLOOR, RNE = ((5, 7, -2, 0), (4, 7, -10, 0)), ((5, 7, -2, 1), (4, 7, -10, 1))


# packed carriers: the finer block where it saves half a round of 256 workgroups; FP32 carriers and rows off 16-byte boundaries: always
@pytest.mark.parametrize("gx,half_round", [(33, 1), (40, 1), (41, 0), (48, 0), (49, 1), (56, 1), (63, 0), (64, 0)])
def test_blocks(gx, half_round):
    M, N = 64 * gx, 1024
    for (qp, qa), K, packed in ((FLOOR, 768, True), (FLOOR, 771, False), (RNE, 768, False)):
        plan = binding.lba_plan_query(M, N, K, qp, qa, 0)
        if plan["tail_blocks"] > 0:
            continue                                           # a mixed grid has blocks of its own
        assert (plan["tile_m"], plan["tile_n"]) == ((64, 64) if packed and not half_round else (32, 64))
    assert binding.lba_plan_query(64 * 64, N, 768, *FLOOR, 0)["tail_blocks"] == 0

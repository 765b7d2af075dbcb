"""Which lane block plain grids of 513 to 1024 workgroups of 64 x 64 take: host logic only (batches, which have no other grids: test_launched_plans_cpu.py)."""
import pytest

from paper_2401_14110_amd import binding

FLOOR, RNE = ((5, 7, -2, 0), (4, 7, -10, 0)), ((5, 7, -2, 1), (4, 7, -10, 1))


# matrices whose grids have no tail of smaller tiles; packed carriers: the finer block where it saves half a round; FP32 carriers: always
@pytest.mark.parametrize("gx,gy,half_round", [(56, 16, 1), (28, 32, 1), (112, 8, 1), (24, 32, 0), (48, 16, 0), (64, 16, 0), (128, 8, 0)])
def test_blocks(gx, gy, half_round):
    for (qp, qa), K, packed in ((FLOOR, 768, True), (FLOOR, 771, True), (RNE, 768, False)):
        plan = binding.lba_plan_query(64 * gx, 64 * gy, K, qp, qa, 0)
        assert plan["tail_blocks"] == 0 and plan["mid_blocks"] == 0
        assert (plan["tile_m"], plan["tile_n"]) == ((64, 64) if packed and not half_round else (32, 64))

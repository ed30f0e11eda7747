"""FP64's automatic tile near one 128x128 tile per CU, where the 64x64 tile had
been taken beyond the sizes it is faster at, and its schedule just above one
wave of 64x64 tiles.  Integer inputs give exact products.
"""
import pytest

from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from tests.test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,blk", [
    (1024, 1792, 4096, 64),      # 448 64x64 tiles: 7/4 of 256 CUs
    (1024, 1792, 4098, 128),
    (1024, 1856, 1792, 64),      # 464
    (1024, 1856, 1794, 128),
    (390, 4160, 1794, 64),       # 455, a seventh of the 128x128 tiles' area padding
    (1664, 1664, 4096, 128),     # 676, none
    (1664, 2048, 64, 64),        # 832: 13/4 of the CUs
    (1664, 2050, 368, 128),      # 858, 23 k-tiles
    (1664, 2050, 370, 64),       # 24
    (1920, 1800, 370, 64),       # 870
    (1664, 2176, 370, 128),      # 884
    (4640, 698, 1794, 64),       # 803, a tenth padding
    (1664, 2048, 1794, 128)])    # 832, none
def test_tile(m, n, k, blk):
    _, plan = check_case(m, n, k, "f64", "f64", dist="int4", ws=R.Workspace("cuda"))
    assert plan.blk_m == blk


@pytest.mark.parametrize("m,n,k,sched", [
    (2050, 1546, 64, S.SK_SCHED_DP), (1664, 1920, 240, S.SK_SCHED_DP),
    (1664, 1920, 242, S.SK_SCHED_DP_1TILE_SK), (1536, 2048, 64, S.SK_SCHED_DP_1TILE_SK)])
def test_schedule_above_one_wave(m, n, k, sched):
    _, plan = check_case(m, n, k, "f64", "f64", dist="int4", ws=R.Workspace("cuda"))
    assert (plan.blk_m, plan.sched) == (64, sched)

"""The automatic split of a few deep tiles on the machine's own slots: equal
pieces (basic Stream-K over that many workgroups), pieces with a shorter last
one (fixed split, placed piece by piece), one workgroup per tile, and the same
calls with the placement switched off; FP64's tile.  Integer inputs give exact
products.
"""
import pytest
import torch

from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from tests.test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ab,ct,m,n,k", [
    ("bf16", "f32", 192, 192, 8192),     # 9 64x64 tiles of 128 k-tiles
    ("f16", "f32", 184, 136, 6680),      # 9 of 105, the last partial
    ("bf16", "bf16", 320, 392, 4096),    # 35 of 64
    ("bf16", "f32", 640, 1024, 4352),    # 40 128x128 tiles of 68
    ("f8e4m3", "bf16", 496, 640, 2064),  # 20 of 17
    ("f8e4m3", "bf16", 1280, 1280, 1024),
    ("f64", "f64", 384, 384, 1024),      # 36 64x64 tiles of 64
    ("f64", "f64", 125, 786, 888),       # 26 of 56, ragged
    ("f64", "f64", 1000, 1000, 514)])    # 256 of 33
def test_few_deep_tiles(ab, ct, m, n, k):
    ws = R.Workspace("cuda")
    got = []
    for flags in (0, S.SK_FLAG_NO_XCD_REMAP):
        C, plan = check_case(m, n, k, ab, ct, dist="int4", cfg=S.make_config(flags=flags), ws=ws)
        assert plan.tiles <= plan.grid <= plan.wg_slots
        got.append(C.view(torch.uint8).cpu())
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("m,n,k,blk", [
    (128, 128, 16, 64), (384, 384, 1024, 64), (126, 786, 888, 64), (2050, 1546, 64, 64),
    (256, 256, 4098, 128), (2048, 2048, 64, 128)])
def test_f64_tile(m, n, k, blk):
    _, plan = check_case(m, n, k, "f64", "f64", dist="int4", ws=R.Workspace("cuda"))
    assert plan.blk_m == blk


@pytest.mark.parametrize("ab,ct,bk", [("bf16", "f32", 64), ("f8e4m3", "bf16", 128)])
def test_grids_of_more_than_two_64_workgroups_per_cu(ab, ct, bk):
    # the caller's grid or split: the kernel that keeps them all resident
    ws = R.Workspace("cuda")
    blk = (64, 64, bk)
    for cfg, g in ((S.make_config(sched="sk", blk=blk, grid=700), 700),
                   (S.make_config(sched="fs", blk=blk, split=3), 3 * 240)):
        _, plan = check_case(1024, 944, 5 * bk - 16, ab, ct, dist="int4", cfg=cfg, ws=ws)
        assert plan.grid == g <= plan.wg_slots
    ws.check()

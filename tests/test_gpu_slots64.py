"""The 16-bit and FP8 64x64 tile has two builds, with two and with more
workgroups per CU: schedules that the caller names are accepted, and exact, with
tile counts between and around the slots of both, where a hybrid's few last
tiles over the deep build's slots would give an owner too many peers.
"""
import pytest
import torch

from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from tests.test_gpu_grouped import check_results, make_batch
from tests.test_gpu_parity import check_case

pytestmark = pytest.mark.gpu

BLK = {"bf16": (64, 64, 64), "f16": (64, 64, 64), "f8e4m3": (64, 64, 128)}


def deep_slots():
    return 2 * torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("ab,ct,tm,tn,iters,sched,split", [
    ("bf16", "f32", 27, 19, 66, "dp1sk", 0),      # 513 tiles: one past the deep build's 512 slots
    ("bf16", "f32", 27, 19, 66, "2tsk", 0),
    ("bf16", "f32", 27, 19, 70, "dp1sk", 70),     # a split that such a plan has no tail for
    ("f16", "f16", 103, 5, 80, "dp1sk", 0),       # 515
    ("f8e4m3", "bf16", 27, 19, 66, "dp1sk", 0),
    ("bf16", "bf16", 29, 53, 66, "dp1sk", 0)])    # 1537
def test_few_tiles_past_the_slots(ab, ct, tm, tn, iters, sched, split):
    cfg = S.make_config(sched=sched, blk=BLK[ab], split=split)
    m, n, k = tm * 64, tn * 64 - 16, iters * BLK[ab][2]
    _, plan = check_case(m, n, k, ab, ct, dist="int4", cfg=cfg, ws=R.Workspace("cuda"), trace=False)
    assert plan.tiles % deep_slots() <= 8 and plan.max_peers <= S.SK_MAX_PEERS


def test_grouped_tail_split_is_ignored_below_a_full_wave():
    # 2 x 270 tiles fit the shallow build's slots: basic Stream-K, nothing to split
    probs = make_batch([(15 * 64, 18 * 64, 192)] * 2, "bf16", "f32", "int4", 3)
    ws = R.Workspace("cuda")
    cfg = S.make_config(sched="dp1sk", blk=BLK["bf16"], split=2)
    plan, raw = R.gemm_grouped([p["d"] for p in probs], cfg=cfg, ws=ws)
    torch.cuda.synchronize()
    ws.check()
    assert plan.tiles == 540 and plan.sched == S.SK_SCHED_SK
    check_results(probs, "bf16", "f32", "int4")


@pytest.mark.parametrize("ab,ct", [("bf16", "f32"), ("f8e4m3", "bf16")])
def test_tiles_that_the_shallow_build_holds_at_once(ab, ct):
    # 600 tiles of 40 k-tiles: one resident workgroup per tile
    cfg = S.make_config(sched="sk", blk=BLK[ab])
    _, plan = check_case(30 * 64, 20 * 64, 40 * BLK[ab][2], ab, ct, dist="int4", cfg=cfg,
                         ws=R.Workspace("cuda"))
    assert plan.grid >= plan.tiles == 600

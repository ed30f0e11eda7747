"""Shares of the 16-bit and FP8 64x64 tile's slots: a plan reports the same
slots whatever its grid, half of them plan a batch for half of the device, and
two launches in flight together on half of them each finish, with exact results.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from tests.test_gpu_grouped import make_batch

pytestmark = pytest.mark.gpu

BLK = {"bf16": (64, 64, 64), "f16": (64, 64, 64), "f8e4m3": (64, 64, 128)}


def reported(d, ab, grid=1):
    st, pl = S.sk_plan(d, S.make_config(sched="sk", blk=BLK[ab], grid=grid))
    S.check(st, "sk_plan")
    return pl.wg_slots


@pytest.mark.parametrize("ab,ct", [("bf16", "f32"), ("f16", "f16"), ("f8e4m3", "bf16")])
def test_reported_slots_do_not_depend_on_the_grid(ab, ct):
    d = make_batch([(640, 640, 8192)], ab, ct, "int4", 1)[0]["d"]
    slots = reported(d, ab)
    assert slots == reported(d, ab, 600) == reported(d, ab, slots)
    st, _ = S.sk_plan(d, S.make_config(sched="sk", blk=BLK[ab], grid=slots + 1))
    assert st == S.SK_ERR_INVALID_VALUE


def test_half_of_the_slots_plan_half_of_the_device():
    # 2 x 50 tiles of 64 k-tiles: Stream-K up to 1.5 workgroups per CU of the share
    probs = make_batch([(640, 320, 4096)] * 2, "bf16", "f32", "int4", 2)
    ds = [p["d"] for p in probs]
    half = reported(ds[0], "bf16") // 2
    st, pl = S.sk_plan(ds, S.make_config(blk=BLK["bf16"], wg_slots=half))
    assert st == S.SK_OK and pl.sched == S.SK_SCHED_SK and pl.grid <= half


@pytest.mark.parametrize("fixup", ["serial", "spread"])
@pytest.mark.parametrize("ab,ct,shapes", [
    ("bf16", "f32", [(512, 512, 16384), (256, 1024, 16384)]),
    ("f8e4m3", "bf16", [(512, 512, 32768), (1024, 256, 32768)])])
def test_two_launches_share_the_slots(ab, ct, shapes, fixup):
    # 64 tiles of 256 k-tiles on 512 workgroups each, in flight on two streams
    runs = []
    for i, (m, n, k) in enumerate(shapes):
        A, B = W.gemm_operands(m, n, k, ab, 11 + i, "int4", fp8_scale=1.0 if ab == "f8e4m3" else None)
        Ad, Bd = A.to("cuda"), B.to("cuda")
        C = torch.zeros((m, n), dtype=W.torch_dtype(ct), device="cuda")
        d = S.make_desc(m, n, k, Ad.tensor, Bd.tensor, C, ab_type=ab, c_type=ct)
        half = reported(d, ab) // 2
        cfg = S.make_config(sched="sk", blk=BLK[ab], grid=half, wg_slots=half, fixup=fixup)
        st, pl = S.sk_plan(d, cfg)
        S.check(st, "sk_plan")
        assert pl.grid == half and pl.sched == S.SK_SCHED_SK
        runs.append(dict(m=m, n=n, k=k, A=A, B=B, Ad=Ad, Bd=Bd, C=C, d=d, cfg=cfg,
                         ws=R.Workspace("cuda", pl.workspace_bytes), stream=torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(12):
        for r in runs:
            S.check(S.sk_gemm(r["d"], r["cfg"], r["ws"].ptr, r["ws"].nbytes, r["stream"].cuda_stream), "sk_gemm")
    for r in runs:
        r["ws"].check(r["stream"].cuda_stream)         # raises if a fixup wait gave up
    for r in runs:
        cref = oracle.gemm(r["m"], r["n"], r["k"], r["A"], r["B"], c_type=ct)
        want = oracle.decode(oracle.round_to(cref, ct), ct)
        assert np.array_equal(r["C"].cpu().double().numpy(), want)

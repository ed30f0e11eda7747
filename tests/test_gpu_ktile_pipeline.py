"""The MAC loops at the k-tile counts where their pipelines change form: fewer
k-tiles than the loads run ahead, odd and even counts (the half-tile loops
take k-tiles in pairs, the FP64 one in fours), the first counts that reach the
loop without edge tests, and a partial last k-tile; interior tiles and tiles
past C's edges.  Integer inputs give exact products, so every result is
bit-exact.
"""
import pytest

from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from tests.test_gpu_parity import check_case

pytestmark = pytest.mark.gpu

BK = {"f64": 16, "f16": 64, "bf16": 64, "f8e4m3": 128}


@pytest.fixture(scope="module")
def ws():
    return R.Workspace("cuda")


@pytest.mark.parametrize("ab,ct", [("f16", "f16"), ("bf16", "f32"), ("f8e4m3", "bf16")])
@pytest.mark.parametrize("ao,bo", [("row", "row"), ("row", "col"), ("col", "row"), ("col", "col")])
@pytest.mark.parametrize("m,n", [(256, 512), (272, 240)])
def test_ktile_counts_and_edges(ab, ct, ao, bo, m, n, ws):
    bk = BK[ab]
    for k in (16, bk, 2 * bk, 3 * bk, 4 * bk + 16, 5 * bk, 6 * bk, 9 * bk - 16):
        check_case(m, n, k, ab, ct, dist="int4", a_order=ao, b_order=bo,
                   cfg=S.make_config(sched="dp", blk=(256, 256, bk)), ws=ws, trace=False)
    # segments that begin and end inside a tile: 2 (or 4) tiles of 7 k-tiles over 5 workgroups
    for fx in ("serial", "spread"):
        check_case(m, n, 7 * bk, ab, ct, dist="int4", a_order=ao, b_order=bo, beta=2.0,
                   cfg=S.make_config(sched="sk", blk=(256, 256, bk), grid=5, fixup=fx), ws=ws)


@pytest.mark.parametrize("ab,ct,blk", [("f16", "f32", 128), ("f16", "f16", 64), ("bf16", "bf16", 128),
                                       ("f8e4m3", "f32", 128), ("f8e4m3", "bf16", 64), ("f64", "f64", 128),
                                       ("f64", "f64", 64)])
@pytest.mark.parametrize("ao,bo", [("row", "row"), ("row", "col"), ("col", "row"), ("col", "col")])
def test_ktile_counts_smaller_tiles(ab, ct, blk, ao, bo, ws):
    bk = BK[ab]
    for (m, n) in ((128, 256), (144, 112)):
        for k in (16, bk, 2 * bk, 3 * bk, 4 * bk + 16, 5 * bk, 8 * bk, 9 * bk - 16, 11 * bk):
            check_case(m, n, k, ab, ct, dist="int4", a_order=ao, b_order=bo,
                       cfg=S.make_config(sched="dp", blk=(blk, blk, bk)), ws=ws, trace=False)
        for fx in ("serial", "spread"):
            check_case(m, n, 7 * bk, ab, ct, dist="int4", a_order=ao, b_order=bo, beta=2.0,
                       cfg=S.make_config(sched="sk", blk=(blk, blk, bk), grid=5, fixup=fx), ws=ws)


@pytest.mark.parametrize("ab,ct", [("f16", "f32"), ("f8e4m3", "bf16")])
@pytest.mark.parametrize("ao,bo", [("row", "row"), ("col", "col")])
def test_many_64_tiles(ab, ct, ao, bo, ws):
    # more than two 64x64 tiles per CU: the data-parallel kernel with two
    # k-tile buffers
    for k in (BK[ab], 5 * BK[ab] + 16):
        check_case(64 * 29 - 16, 64 * 27, k, ab, ct, dist="int4", a_order=ao, b_order=bo,
                   cfg=S.make_config(sched="dp", blk=(64, 64, BK[ab])), ws=ws, trace=False)

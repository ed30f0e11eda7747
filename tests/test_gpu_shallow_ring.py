"""The two-buffer MAC loop of the 16-bit 64x64 tile (more than two workgroups
per CU) at the k-tile counts where its loads change form: fewer k-tiles than the
loads run ahead, the first counts that reach the loop without edge tests, a
partial last k-tile; whole tiles and segments that begin and end inside one.
Integer inputs give exact products.
"""
import pytest

from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from tests.test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    return R.Workspace("cuda")


@pytest.mark.parametrize("ab,ct", [("f16", "f16"), ("bf16", "f32")])
@pytest.mark.parametrize("ao,bo", [("row", "row"), ("row", "col"), ("col", "row"), ("col", "col")])
def test_ktile_counts(ab, ct, ao, bo, ws):
    m, n = 64 * 29 - 16, 64 * 27 - 24
    for k in (16, 64, 120, 128, 192, 256, 328, 384):
        _, plan = check_case(m, n, k, ab, ct, dist="int4", a_order=ao, b_order=bo,
                             cfg=S.make_config(sched="dp", blk=(64, 64, 64)), ws=ws, trace=False)
        assert plan.grid == 783
    for fx, grid in (("serial", 700), ("spread", 1000)):
        _, plan = check_case(64 * 9 - 8, 64 * 8, 64 * 41, ab, ct, dist="int4", a_order=ao, b_order=bo, beta=2.0,
                             cfg=S.make_config(sched="sk", blk=(64, 64, 64), grid=grid, fixup=fx), ws=ws)
        assert plan.grid == grid

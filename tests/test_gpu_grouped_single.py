"""A grouped call of one problem under the default configuration: the
workspace that sk_plan and sk_workspace_size ask for (they size sk_gemm and
sk_gemm_grouped alike) is enough for it, to the byte, and the result is exact.
"""
import pytest
import torch

from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from tests.test_gpu_grouped import check_results, make_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ab,ct,m,n,k", [
    ("f64", "f64", 128, 128, 512),       # few 64x64 tiles, split
    ("f64", "f64", 1000, 1000, 514),     # 256 of them, one workgroup each
    ("f64", "f64", 1500, 1000, 400),     # more of them than CUs
    ("f64", "f64", 256, 256, 4098),      # 128x128 tiles
    ("bf16", "f32", 192, 192, 8192),
    ("f16", "f16", 640, 1024, 4352),
    ("f8e4m3", "bf16", 496, 640, 2064)])
def test_one_problem_fits_the_planned_workspace(ab, ct, m, n, k):
    probs = make_batch([(m, n, k)], ab, ct, "int4", 5)
    st, need = S.sk_workspace_size(probs[0]["d"], None)
    S.check(st, "sk_workspace_size")
    ws = R.Workspace("cuda", need)
    plan, raw = R.gemm_grouped([probs[0]["d"]], ws=ws)
    assert plan.workspace_bytes == need == ws.nbytes
    torch.cuda.synchronize()
    ws.check()
    check_results(probs, ab, ct, "int4")

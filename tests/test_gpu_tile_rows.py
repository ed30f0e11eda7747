"""C's rows as the tile epilogue writes them: rows that end inside a vector,
rows that are not vector-aligned, tiles past both edges, with and without old
values of C, in a buffer with wider rows whose rest must stay untouched.
Integer inputs give exact sums, so every result is bit-exact.
"""
import ctypes

import pytest
import torch

from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import streamk as S
from workloads import torch_dtype

pytestmark = pytest.mark.gpu

BK = {"f16": 64, "bf16": 64, "f8e4m3": 128}


@pytest.mark.parametrize("ab,ct", [("f16", "f16"), ("f16", "f32"), ("bf16", "bf16"), ("f8e4m3", "f32")])
@pytest.mark.parametrize("blk", [64, 128, 256])
@pytest.mark.parametrize("m,n,pad", [(256, 512, 0), (255, 510, 2), (257, 259, 5), (70, 301, 0), (1, 1, 7)])
def test_rows_of_c(ab, ct, blk, m, n, pad):
    k = BK[ab] + 16
    gen = torch.Generator().manual_seed(m + n)

    def ints(*shape):
        return torch.randint(-4, 5, shape, generator=gen).float()
    A, B, C0 = ints(m, k), ints(n, k), ints(m, n)
    dt = torch_dtype(ct)
    Ad, Bd = A.to(torch_dtype(ab)).cuda(), B.to(torch_dtype(ab)).cuda()
    for beta in (0.0, 2.0):
        want = (A.double() @ B.double().t() + beta * C0.double()).float().to(dt)
        buf = torch.full((m + 1, n + pad), 77.0, dtype=dt)
        buf[:m, :n] = C0.to(dt)
        whole = buf.clone()
        whole[:m, :n] = want
        buf = buf.cuda()
        d = S.make_desc(m, n, k, Ad, Bd, buf, ab_type=ab, c_type=ct, b_order="col", beta=beta, ldc=n + pad)
        cfg = S.make_config(sched="dp", blk=(blk, blk, BK[ab]))
        pl = S.sk_plan_t()
        assert S.lib().sk_plan(ctypes.pointer(d), 1, ctypes.byref(cfg), ctypes.byref(pl)) == 0
        w = R.Workspace("cuda", pl.workspace_bytes)
        assert S.lib().sk_gemm(ctypes.byref(d), ctypes.byref(cfg), ctypes.c_void_p(w.ptr), w.nbytes, None) == 0
        torch.cuda.synchronize()
        assert torch.equal(buf.cpu().float(), whole.float()), (beta,)

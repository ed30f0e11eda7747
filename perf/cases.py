"""Performance cases of the Stream-K GEMM library.

Single GEMMs run through ``sk_gemm`` with a descriptor and a workspace the
program keeps (the README's usage) or through ``runtime.gemm``, which builds
the descriptor and plans on each call; batches through ``sk_gemm_grouped``;
request streams through ``serve.Server``.  Every call uses the library's
default configuration.  Sizes come from the workloads the benchmark and the
tests run: the geometry sweep (m, n, k log-uniform in [128, 8192]), the
FP64 example problem, the precision set, the grouped batch and the serving
mix, plus ragged sizes of the same range.
"""
from __future__ import annotations

import math
import random

import torch

import workloads as W
from paper_2301_03598_amd import runtime as R
from paper_2301_03598_amd import serve as V
from paper_2301_03598_amd import streamk as S

# elements per 16 bytes: what a contiguous extent of A or B is a multiple of
_VEC = {"f64": 2, "f16": 8, "bf16": 8, "f8e4m3": 16}


def _gemm(name, ab, ct, m, n, k, dist, a_order="row", b_order="row", beta=0.0, call="handle"):
    return {"name": name, "kind": "gemm", "ab": ab, "ct": ct, "m": m, "n": n, "k": k, "dist": dist,
            "a_order": a_order, "b_order": b_order, "beta": beta, "call": call}


def listed():
    return [
        # one small request of the serving mix on its own: latency and launch
        # cost, through the convenience call
        _gemm("f16_small_call", "f16", "f32", 200, 136, 520, "normal", call="runtime"),
        # the FP64 example problem: 9 output tiles for 256 CUs
        _gemm("f64_384x384x1024", "f64", "f64", 384, 384, 1024, "uniform"),
        # a thin layer: few rows against a k-contiguous (transposed) weight
        _gemm("bf16_thin_rows", "bf16", "bf16", 129, 4096, 2048, "normal", b_order="col"),
        # C += A^T B with a ragged C (a weight gradient added to what is there)
        _gemm("bf16_accumulate_ragged", "bf16", "f32", 1736, 969, 2120, "normal",
              a_order="col", b_order="col", beta=1.0),
        # few output tiles, deep k (a split-k reduction): 128 flops a byte
        _gemm("bf16_256x256x65536", "bf16", "bf16", 256, 256, 65536, "normal"),
        # the precision set's wide shape: one layer's product in FP8
        _gemm("f8_4096x1024x4096", "f8e4m3", "bf16", 4096, 1024, 4096, "normal"),
        # an FP64 problem of the sweep's middle
        _gemm("f64_2050x1546x1034", "f64", "f64", 2050, 1546, 1034, "uniform"),
        # 24 problems of the geometry sweep, one call each
        {"name": "f16_sweep_24", "kind": "sweep", "ab": "f16", "ct": "f32", "count": 24, "shape_seed": 1},
        # a batch of uneven GEMMs in one grouped launch
        {"name": "bf16_grouped_64", "kind": "grouped", "ab": "bf16", "ct": "bf16", "count": 64,
         "shape_seed": 3},
        # a burst of mixed requests drained by the server (BF16 and FP16)
        {"name": "serve_burst_48", "kind": "serve", "count": 48, "shape_seed": 4},
        # the large square shape, in both narrow types
        _gemm("bf16_8192", "bf16", "bf16", 8192, 8192, 8192, "normal"),
        _gemm("f8_8192", "f8e4m3", "bf16", 8192, 8192, 8192, "normal"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, lo, hi, mult):
    return max(mult, int(round(_log_uniform(rng, lo, hi) / mult)) * mult)


def draw(rng: random.Random):
    kind = rng.choices(["gemm", "sweep", "grouped", "serve"], [8, 1, 1, 1])[0]
    if kind == "sweep":
        return {"kind": "sweep", "ab": rng.choice(["f16", "bf16"]), "ct": "f32",
                "count": rng.randint(4, 24), "shape_seed": rng.randint(10, 10 ** 6)}
    if kind == "grouped":
        return {"kind": "grouped", "ab": "bf16", "ct": rng.choice(["bf16", "f32"]),
                "count": int(_log_uniform(rng, 4, 64)), "shape_seed": rng.randint(10, 10 ** 6)}
    if kind == "serve":
        return {"kind": "serve", "count": int(_log_uniform(rng, 4, 32)),
                "shape_seed": rng.randint(10, 10 ** 6)}
    ab = rng.choice(["f16", "f16", "bf16", "bf16", "f8e4m3", "f64"])
    ct = {"f64": ["f64"], "f16": ["f32", "f16"], "bf16": ["bf16", "f32"], "f8e4m3": ["bf16", "f32"]}[ab]
    a_order = rng.choice(["row", "row", "col"])
    b_order = rng.choice(["row", "row", "col"])
    v = _VEC[ab]
    hi = 4096 if ab == "f64" else 8192
    # only the contiguous extents of A and B need whole 16-byte vectors
    m = _size(rng, 96, hi, v if a_order == "col" else 1)
    n = _size(rng, 96, hi, v if b_order == "row" else 1)
    k = _size(rng, 128, hi, v)
    if rng.random() < 0.1 and ab != "f64":       # few tiles, deep k
        m = _size(rng, 128, 512, v)
        n = _size(rng, 128, 512, v)
        k = _size(rng, 8192, 65536, v)
    return {"kind": "gemm", "ab": ab, "ct": rng.choice(ct), "m": m, "n": n, "k": k,
            "dist": rng.choice(["normal", "uniform"]), "a_order": a_order, "b_order": b_order,
            "beta": rng.choice([0.0, 0.0, 0.0, 1.0]), "call": rng.choice(["handle", "handle", "runtime"])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _fill(shape, dist, gen):
    t = torch.empty(shape, dtype=torch.float32, device="cuda")
    return t.uniform_(-1.0, 1.0, generator=gen) if dist == "uniform" else t.normal_(0.0, 1.0, generator=gen)


def _operand(rows, cols, ab, order, dist, gen):
    """A stored matrix: the tensor in its storage order and (FP8) its scale."""
    shape = (rows, cols) if order == "row" else (cols, rows)
    if ab == "f64":
        t = torch.empty(shape, dtype=torch.float64, device="cuda")
        t = t.uniform_(-1.0, 1.0, generator=gen) if dist == "uniform" else t.normal_(0.0, 1.0, generator=gen)
        return t, 1.0
    x = _fill(shape, dist, gen)
    if ab == "f8e4m3":
        scale = float(x.abs().max()) / W.FP8_E4M3_MAX
        return (x / scale).clamp_(-W.FP8_E4M3_MAX, W.FP8_E4M3_MAX).to(torch.float8_e4m3fn), scale
    return x.to(W.torch_dtype(ab)), 1.0


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _gemm_inputs(case, seed):
    g = _gen(seed)
    a, sa = _operand(case["m"], case["k"], case["ab"], case["a_order"], case["dist"], g)
    b, sb = _operand(case["k"], case["n"], case["ab"], case["b_order"], case["dist"], g)
    c0 = None
    if case["beta"] != 0.0:
        c0 = _operand(case["m"], case["n"], case["ct"], "row", case["dist"], g)[0]
    return a, sa, b, sb, c0


def _shapes(case):
    if case["kind"] == "sweep":
        return W.sweep_shapes(case["count"], case["shape_seed"])
    if case["kind"] == "grouped":
        return W.grouped_shapes(case["count"], case["shape_seed"])
    raise ValueError(case["kind"])


def _trace(case):
    return W.serving_trace(rate_per_s=20000.0, duration_s=10.0, seed=case["shape_seed"],
                           max_requests=case["count"])


def _many_inputs(case, seed):
    g = _gen(seed)
    dist = "uniform" if case["kind"] == "sweep" else "normal"
    return [(_operand(m, k, case["ab"], "row", dist, g)[0], _operand(k, n, case["ab"], "row", dist, g)[0])
            for (m, n, k) in _shapes(case)]


# elements of one operand pool: the largest request's operand and room to move
_POOL = 160 << 20


def _serve_inputs(case, seed):
    g = _gen(seed)
    pools = {}
    for dt in ("bf16", "f16"):
        pools[dt] = torch.empty(_POOL, dtype=W.torch_dtype(dt), device="cuda")
        pools[dt].normal_(0.0, 1.0, generator=g)
    reqs = V.make_requests(_trace(case), pools, seed=seed)
    for r in reqs:
        r.arrival = 0.0
    return pools, reqs


def _stream():
    return torch.cuda.current_stream().cuda_stream


def prepare(case, seed):
    if case["kind"] == "gemm":
        a, sa, b, sb, c0 = _gemm_inputs(case, seed)
        m, n, k, ab, ct = case["m"], case["n"], case["k"], case["ab"], case["ct"]
        c = torch.empty((m, n), dtype=W.torch_dtype(ct), device="cuda")
        st = {"case": case, "a": a, "b": b, "c": c, "c0": c0, "ws": R.Workspace("cuda")}
        d = S.make_desc(m, n, k, a, b, c, ab_type=ab, c_type=ct, a_order=case["a_order"],
                        b_order=case["b_order"], beta=case["beta"], a_scale=sa, b_scale=sb)
        status, plan = S.sk_plan(d)
        S.check(status, "sk_plan")
        st["ws"].ensure(plan.workspace_bytes)
        if case["call"] == "handle":
            st["desc"] = d
        else:
            st["A"] = W.Operand(a, m, k, ab, case["a_order"], a.shape[1], sa)
            st["B"] = W.Operand(b, k, n, ab, case["b_order"], b.shape[1], sb)
        return st
    if case["kind"] == "sweep":
        ops = _many_inputs(case, seed)
        outs, descs, need = [], [], 256
        for (m, n, k), (a, b) in zip(_shapes(case), ops):
            c = torch.empty((m, n), dtype=W.torch_dtype(case["ct"]), device="cuda")
            d = S.make_desc(m, n, k, a, b, c, ab_type=case["ab"], c_type=case["ct"])
            status, plan = S.sk_plan(d)
            S.check(status, "sk_plan")
            need = max(need, plan.workspace_bytes)
            outs.append(c)
            descs.append(d)
        return {"case": case, "ops": ops, "outs": outs, "descs": descs, "ws": R.Workspace("cuda", need)}
    if case["kind"] == "grouped":
        ops = _many_inputs(case, seed)
        outs = [torch.empty((m, n), dtype=W.torch_dtype(case["ct"]), device="cuda") for (m, n, _) in _shapes(case)]
        descs = [S.make_desc(m, n, k, a, b, c, ab_type=case["ab"], c_type=case["ct"])
                 for (m, n, k), (a, b), c in zip(_shapes(case), ops, outs)]
        ws = R.Workspace("cuda")
        # the first launch plans, sizes the workspace and pins the descriptors
        _, pinned = R.gemm_grouped(descs, ws=ws)
        return {"case": case, "ops": ops, "outs": outs, "pinned": pinned, "ws": ws}
    pools, reqs = _serve_inputs(case, seed)
    return {"case": case, "pools": pools, "reqs": reqs, "server": V.Server(pools, out_bytes=4 << 30)}


def run(state):
    case = state["case"]
    if case["kind"] == "gemm":
        if state["c0"] is not None:
            state["c"].copy_(state["c0"])
        if case["call"] == "handle":
            ws = state["ws"]
            S.check(S.sk_gemm(state["desc"], None, ws.ptr, ws.nbytes, _stream()), "sk_gemm")
        else:
            R.gemm(case["m"], case["n"], case["k"], state["A"], state["B"], state["c"], c_type=case["ct"],
                   beta=case["beta"], ws=state["ws"])
        return state["c"]
    if case["kind"] == "sweep":
        ws, s = state["ws"], _stream()
        for d in state["descs"]:
            S.check(S.sk_gemm(d, None, ws.ptr, ws.nbytes, s), "sk_gemm")
        return state["outs"]
    if case["kind"] == "grouped":
        ws = state["ws"]
        S.check(S.sk_gemm_grouped((state["pinned"].data_ptr(), case["count"]), None, ws.ptr, ws.nbytes, _stream()),
                "sk_gemm_grouped")
        return state["outs"]
    server = state["server"]
    server.run(state["reqs"])
    return [server.output(r) for r in state["reqs"]]


# ---------------------------------------------------------------------------
# cost and 64-bit values
# ---------------------------------------------------------------------------

def _cost(m, n, k, ab, ct, beta=0.0):
    eb, cb = W.DTYPE_BYTES[ab], W.DTYPE_BYTES[ct]
    return (m * k + k * n) * eb + m * n * cb * (2 if beta != 0.0 else 1), 2.0 * m * n * k


def work(case):
    if case["kind"] == "gemm":
        parts = [_cost(case["m"], case["n"], case["k"], case["ab"], case["ct"], case["beta"])]
    elif case["kind"] == "serve":
        parts = [_cost(r.m, r.n, r.k, r.dtype, "f32") for r in _trace(case)]
    else:
        parts = [_cost(m, n, k, case["ab"], case["ct"]) for (m, n, k) in _shapes(case)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def exact(case, seed):
    if case["kind"] == "gemm":
        a, sa, b, sb, c0 = _gemm_inputs(case, seed)
        a64 = a.double() if case["a_order"] == "row" else a.double().t()
        b64 = b.double() if case["b_order"] == "row" else b.double().t()
        # the library holds the FP8 scales in 32 bits
        sa = float(torch.tensor(sa, dtype=torch.float32))
        sb = float(torch.tensor(sb, dtype=torch.float32))
        out = torch.matmul(a64, b64) * (sa * sb)
        return out if c0 is None else out + case["beta"] * c0.double()
    if case["kind"] == "serve":
        pools, reqs = _serve_inputs(case, seed)
        outs = []
        for r in reqs:
            p = pools[r.dtype]
            a = p[r.a_off:r.a_off + r.m * r.k].view(r.m, r.k)
            b = p[r.b_off:r.b_off + r.k * r.n].view(r.k, r.n)
            outs.append(torch.matmul(a.double(), b.double()))
        return outs
    return [torch.matmul(a.double(), b.double()) for (a, b) in _many_inputs(case, seed)]

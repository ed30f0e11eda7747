"""The kernels issue their global -> LDS loads as text, which the compiler's
hazard handling does not see into.  A scalar register that a vector instruction
wrote (the readlane of a spilled one, say) may be read by a vector-memory
instruction after five wait states at the earliest, m0 by such a load one after it
was written.  The machine code of the built library is checked for both, along
every path into each load.
"""
import concurrent.futures as cf
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2301_03598_amd import streamk as S

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# vector instructions whose second operand is a scalar destination
SECOND = ("v_mad_u64", "v_mad_i64", "v_add_co", "v_sub_co", "v_subrev_co", "v_addc_co", "v_subb", "v_div_scale")
END = ("s_branch", "s_endpgm", "s_setpc_b64")


def sregs(op):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", op)
    if not m:
        return {"m0"} if op == "m0" else set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def split(line):
    name, _, rest = line.split("//")[0].strip().partition(" ")
    return name, re.findall(r"[\w.]+\[\d+:\d+\]|[\w.]+", rest)


def written(name, ops):
    """Scalar registers that the instruction writes."""
    if not ops:
        return set()
    if name.startswith("v_"):
        return sregs(ops[0]) or (sregs(ops[1]) if name.startswith(SECOND) else set())
    return sregs(ops[0]) if ops[0] == "m0" else set()


def hazards(text):
    """(loads found, the offending pairs) of a listing."""
    lines = text.splitlines()
    func, jumps, start = [], {}, 0
    for i, l in enumerate(lines):
        if l.startswith("<") and not re.match(r"<L\d+>:", l):
            start = i
        func.append(start)
        if "branch" in l:
            jumps.setdefault((start, split(l)[1][-1]), []).append(i)
    bad = []

    def back(i, load, regs, states):
        # everything that can run up to and including line i before the load,
        # `states` wait states already between
        while states < 5 and i > func[load]:
            if lines[i].startswith("<"):
                for j in jumps.get((func[load], lines[i][1:lines[i].index(">")]), []):
                    back(j - 1, load, regs, states + 1)
            else:
                name, ops = split(lines[i])
                if name in END:
                    return
                hit = written(name, ops) & regs
                if hit and (name.startswith("v_") or states < 1):
                    bad.append((lines[i].strip(), lines[load].strip()))
                if hit:
                    return
                states += int(ops[0], 0) + 1 if name == "s_nop" else 1
            i -= 1

    loads = [i for i, l in enumerate(lines) if l.lstrip().startswith("buffer_load") and " lds" in l]
    for i in loads:
        regs = {r for o in split(lines[i])[1] for r in sregs(o)}
        back(i - 1, i, regs, 0)
        back(i - 1, i, {"m0"}, 0)
    return len(loads), bad


LOAD = "\ts_mov_b32 m0, s72\n\ts_nop 0\n\tbuffer_load_dwordx4 v4, s[40:43], s59 offen lds\n"


@pytest.mark.parametrize("text,count", [
    ("<f>:\n\ts_mov_b32 s41, s2\n" + LOAD, 0),
    ("<f>:\n\tv_readlane_b32 s41, v9, 3\n" + LOAD, 1),
    ("<f>:\n\tv_readlane_b32 s44, v9, 3\n" + LOAD, 0),
    ("<f>:\n\tv_mad_u64_u32 v[2:3], s[58:59], v1, v2, v[4:5]\n\ts_add_i32 s1, s1, 1\n\ts_nop 0\n" + LOAD, 1),
    ("<f>:\n\tv_readfirstlane_b32 s59, v9\n\ts_nop 2\n" + LOAD, 0),
    ("<f>:\n\tv_readlane_b32 s40, v9, 3\n\ts_branch L1\n<L0>:\n\ts_nop 7\n<L1>:\n" + LOAD, 1),
    ("<f>:\n\tv_readlane_b32 s40, v9, 3\n\ts_branch L2\n<L1>:\n" + LOAD + "<L2>:\n\ts_endpgm\n", 0),
    ("<f>:\n\ts_mov_b32 m0, s72\n\tbuffer_load_dwordx4 v4, s[40:43], 0 offen lds\n", 1)])
def test_the_check_itself(text, count):
    loads, bad = hazards(text)
    assert loads == 1 and len(bad) == count, bad


@pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(S.LIB_PATH)),
                    reason="needs the built library and the compiler's listing tool")
def test_built_kernels_have_the_wait_states(tmp_path):
    shutil.copy(S.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)

    def check(path):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands", path],
                             check=True, capture_output=True, text=True)
        return hazards(out.stdout)
    with cf.ThreadPoolExecutor(4) as ex:
        found = list(ex.map(check, sorted(glob.glob(str(tmp_path / "lib.so.*gfx950")))))
    assert sum(n for n, _ in found) > 1000
    bad = [b for _, lst in found for b in lst]
    assert not bad, f"{len(bad)} hazards, first {bad[:3]}"

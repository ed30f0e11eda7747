"""Write the kernel-instance translation units (one per dtype x tile x
operand contiguity) and the lookup table that selects among them.  Splitting
the instances this finely lets hipcc compile them in parallel.

Run from anywhere: python paper_2301_03598_amd/csrc/gen_instances.py
"""
import os

HERE = os.path.dirname(os.path.abspath(__file__))

# (name, Dt enumerator, ab_type enumerator, tiles); a tile is its edge, or
# (edge, waves per workgroup) where that is not four.  The 256x256 tiles run
# eight waves, two per SIMD in two groups half a phase apart (mac_loop_pp):
# 8192^3 BF16 881 -> 727 us, FP8 583 -> 397.
DTYPES = [("f64", "F64", "SK_F64", [128, 64]),
          ("f16", "F16", "SK_F16", [(256, 8), 128, 64]),
          ("bf16", "BF16", "SK_BF16", [(256, 8), 128, 64]),
          ("f8", "F8", "SK_F8_E4M3", [(256, 8), 128, 64])]


LAYOUTS = [("kk", "true", "true"), ("kn", "true", "false"), ("nk", "false", "true"), ("nn", "false", "false")]


def tile_waves(t):
    return t if isinstance(t, tuple) else (t, 4)


def unit(dt, enum, tile, lay, akc, bkc, nw=4):
    w = "" if nw == 4 else f", {nw}"
    waves = "" if nw == 4 else f" ({nw} waves)"
    return f"""// Generated by gen_instances.py: {enum} inputs, {tile}x{tile} tiles{waves}, A {'k' if akc == 'true' else 'm'}-contiguous,
// B {'k' if bkc == 'true' else 'n'}-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {{
KernelEntry pick_{dt}_{tile}_{lay}(const KernelKey &k) {{
    return k.grouped ? entry<Dt::{enum}, {tile}, {tile}, {akc}, {bkc}, true{w}>(k)
                     : entry<Dt::{enum}, {tile}, {tile}, {akc}, {bkc}, false{w}>(k);
}}
}}  // namespace sk
"""


def table():
    decls, cases = [], []
    for dt, enum, ab, tiles in DTYPES:
        for tile, _ in map(tile_waves, tiles):
            for lay, akc, bkc in LAYOUTS:
                decls.append(f"KernelEntry pick_{dt}_{tile}_{lay}(const KernelKey &k);")
                cases.append(f"    if (k.ab_type == {ab} && k.bm == {tile} && k.bn == {tile} && k.a_kc == {akc} && "
                             f"k.b_kc == {bkc}) return pick_{dt}_{tile}_{lay}(k);")
    return ("// Generated by gen_instances.py: the kernel-instance lookup.\n#include \"sk_internal.h\"\n\n"
            "namespace sk {\n" + "\n".join(decls) + "\n\nKernelEntry find_kernel(const KernelKey &k) {\n" +
            "\n".join(cases) + "\n    return KernelEntry{nullptr, nullptr};\n}\n}  // namespace sk\n")


def expected():
    """File name -> content of every generated unit and of the table."""
    out = {}
    for dt, enum, ab, tiles in DTYPES:
        for tile, nw in map(tile_waves, tiles):
            for lay, akc, bkc in LAYOUTS:
                out[f"inst_{dt}_{tile}_{lay}.hip"] = unit(dt, enum, tile, lay, akc, bkc, nw)
    out["sk_table.cpp"] = table()
    return out


def main():
    for f in os.listdir(HERE):
        if f.startswith("inst_") and f.endswith(".hip"):
            os.remove(os.path.join(HERE, f))
    for name, text in expected().items():
        with open(os.path.join(HERE, name), "w") as fh:
            fh.write(text)


if __name__ == "__main__":
    main()

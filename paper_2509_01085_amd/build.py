"""Build libbsa.so (HIP, gfx950) in-tree with hipcc.  `python -m paper_2509_01085_amd.build`."""
from __future__ import annotations

import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libbsa.so")
SOURCES = [
    "bsa_api.hip",
    "bsa_pool_prune.hip",
    "bsa_select.hip",
    "bsa_attn_generic.hip",
    "bsa_attn_fwd.hip",
    "bsa_attn_pipe.hip",
    "bsa_attn_dkv.hip",
    "bsa_probe.hip",
]
# -ffp-contract=off: the decision kernels fix every rounding; packed-fp32 ops are disabled
# on the test machines (some forms have produced wrong results).
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
]
# bsa_attn_fwd: its wavefronts choose between code paths on scalars.  Structured like divergent branches, such paths would keep
# separate registers for what they have in common, and moves between them.
EXTRA_FLAGS = {"bsa_attn_fwd.hip": ["-mllvm", "-structurizecfg-skip-uniform-regions"]}

# Kernels that keep values in accumulation registers which inline assembly names: the compiler does not know of them, so it may
# have none of its own there.
NAMED_ACCUMULATORS = {"bsa_attn_fwd.hip": "fwd_walk_kernel"}


def foreign_accumulators(assembly: str, kernel: str):
    """Instructions of the kernel's instances that name an accumulation register and are not inline assembly, and the number
    of instances."""
    found, instances, inside, inline = [], 0, False, False
    for line in assembly.splitlines():
        if re.match(r"_Z\w*:", line):
            inside, inline = kernel in line.split(":")[0], False
            instances += inside
        elif line.startswith(".Lfunc_end"):
            inside = False
        elif "#ASMSTART" in line or "#ASMEND" in line:
            inline = "#ASMSTART" in line
        elif inside and not inline and re.search(r"(?<![\w.@$])a(\d+\b|\[)", line.split(";")[0]):
            found.append(line.strip())
    return found, instances


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = True, out: str = LIB, extra_flags=()) -> str:
    """Compile every source and link `out`.  `extra_flags` (e.g. -DNAME=value tuning macros)
    go to every compile; objects of such variant builds live in their own folder."""
    global OBJ
    obj_dir = OBJ if out == LIB else OBJ + "_" + os.path.basename(out).replace(".", "_")
    os.makedirs(obj_dir, exist_ok=True)

    def comp(src):
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [hipcc(), *FLAGS, *EXTRA_FLAGS.get(src, ()), *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        noise = "is not a recognized feature for this target"
        err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
        if r.returncode:
            raise RuntimeError(f"hipcc failed for {src}:\n{err}")
        if err.strip():
            print(err, file=sys.stderr)
        return obj

    def check(src):
        cmd = [hipcc(), *FLAGS, *EXTRA_FLAGS.get(src, ()), *extra_flags, "-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", "-"]
        r = subprocess.run(cmd, capture_output=True, text=True)
        found, instances = foreign_accumulators(r.stdout, NAMED_ACCUMULATORS[src])
        if r.returncode or found or not instances:
            raise RuntimeError(f"{src}: the compiler uses accumulation registers that the source names: {found[:5]}" if found else
                               f"{src}: no assembly of {NAMED_ACCUMULATORS[src]}:\n{r.stderr[-2000:]}")

    with ThreadPoolExecutor(max_workers=8) as ex:
        checks = [ex.submit(check, src) for src in NAMED_ACCUMULATORS]
        objs = list(ex.map(comp, SOURCES))
        for c in checks:
            c.result()
    LIB_OUT = out
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_OUT, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB_OUT)
    return LIB_OUT


if __name__ == "__main__":
    # python -m paper_2509_01085_amd.build [-o other.so] [-DFLAG ...]
    argv = sys.argv[1:]
    out = LIB
    if "-o" in argv:
        k = argv.index("-o")
        out = os.path.abspath(argv[k + 1])
        del argv[k:k + 2]
    build(out=out, extra_flags=tuple(argv))

"""Builds libsvg2_hip.so (the C-ABI library) for gfx950 with hipcc, in-tree, and libsvg2_hip_test.so: the same with the entry points
that only the tests call (SVG2_TEST_HOOKS)."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsvg2_hip.so")
TEST_LIB = os.path.join(HERE, "libsvg2_hip_test.so")
SOURCES = ["svg2_api.hip", "svg2_permute.hip", "svg2_select.hip", "svg2_kmeans.hip", "svg2_attn.hip", "svg2_fp8.hip",
           "svg2_diag.hip"]
TEST_HOOKS = ["svg2_diag.hip"]              # sources with entry points for the tests
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-result", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def build(verbose: bool = False) -> str:
    """Compile every source (always; hipcc cross-compiles without a GPU) and link the shared library."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    for s, define in [(s, []) for s in SOURCES] + [(s, ["-DSVG2_TEST_HOOKS"]) for s in TEST_HOOKS]:
        obj = os.path.join(objdir, s.replace(".hip", "_test.o" if define else ".o"))
        cmd = ["hipcc", *FLAGS, *define, "-c", os.path.join(CSRC, s), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((s, obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    objs = []
    for s, obj, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip() != "1 warning generated when compiling for host.")
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (s, out))
        if verbose and out.strip():
            print(out)
        objs.append(obj)
    plain, hooked = objs[:len(SOURCES)], objs[len(SOURCES):]
    replaced = [o.replace("_test.o", ".o") for o in hooked]
    for lib, parts in ((LIB, plain), (TEST_LIB, [o for o in plain if o not in replaced] + hooked)):
        tmp = lib + ".tmp.%d" % os.getpid()
        subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *parts])
        os.replace(tmp, lib)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

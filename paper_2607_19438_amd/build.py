"""Build the gfx950 shared library ``libqgemm.so`` in-tree with hipcc.

Usage: ``python -m paper_2607_19438_amd.build [--verbose]``.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqgemm.so")
SOURCES = [os.path.join(CSRC, f) for f in ("qgemm_api.hip", "moe_direct.hip")]
DEPS = SOURCES + [os.path.join(CSRC, f) for f in ("qgemm_kernels.hpp", "qgemm_aux.hpp", "qgemm_smallm.hpp", "moe_direct.hpp",
                                                  "moe_direct_api.hpp", "tile_rules.hpp", "attn_kernels.hpp")] + [
    os.path.join(os.path.dirname(HERE), "include", "qgemm.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++20",
    "-fPIC",
    # no packed-fp32 VALU instructions in any device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False, extra=None) -> str:
    """Compile every source (side by side, one object each) and link the library. All of it in a folder of
    its own beside the library, which then replaces the old one in one step: builds may run at once."""
    with tempfile.TemporaryDirectory(prefix="build-", dir=os.path.dirname(LIB)) as tmp:
        objs = [os.path.join(tmp, os.path.basename(src) + ".o") for src in SOURCES]
        new = os.path.join(tmp, os.path.basename(LIB))
        cmds = [[HIPCC, *FLAGS, *(extra or []), "-c", src, "-o", obj] for src, obj in zip(SOURCES, objs)]
        link = [HIPCC, f"--offload-arch={ARCH}", "-shared", *objs, "-o", new]
        if verbose:
            for cmd in [*cmds, link]:
                print(" ".join(cmd), flush=True)
        procs = [subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for cmd in cmds]
        outs = [p.communicate()[0] for p in procs]
        rcs = [p.returncode for p in procs]
        if not any(rcs):
            res = subprocess.run(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            outs.append(res.stdout)
            rcs.append(res.returncode)
        out = "\n".join(l for l in "".join(outs).splitlines() if "not a recognized feature" not in l)
        if any(rcs):
            raise RuntimeError(f"hipcc failed ({rcs}):\n{out}")
        if verbose and out.strip():
            print(out)
        os.replace(new, LIB)
    return LIB


if __name__ == "__main__":
    v = "--verbose" in sys.argv
    extra = ["-Rpass-analysis=kernel-resource-usage"] if "--resources" in sys.argv else None
    print(build(verbose=v or bool(extra), extra=extra))

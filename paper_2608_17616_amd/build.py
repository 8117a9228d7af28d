"""Build the HIP library libmone_ttl.so for gfx950, in the package directory.

    python -m paper_2608_17616_amd.build [--verbose]
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SOURCES = [os.path.join(PKG, "csrc", f) for f in
           ("mone_ttl.hip", "mone_swiglu.hip", "swiglu_step.hip", "attention.hip")]
DEPENDS = SOURCES + [os.path.join(PKG, "csrc", f) for f in
                     ("kernels.hpp", "main_loop.inc", "host_common.hpp", "swiglu_kernels.hpp",
                      "swiglu_step.hpp", "attention.hpp")] + [
                     os.path.join(ROOT, "include", f) for f in ("mone_ttl.h", "mone_swiglu.h")]
LIB = os.path.join(PKG, "libmone_ttl.so")
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build the HIP library)")


def build(verbose: bool = False, extra_flags: list[str] | None = None) -> str:
    """One compilation per source file, in parallel, then the link."""
    flags = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
             # keep the compiler from emitting packed fp32 arithmetic
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-I", os.path.join(ROOT, "include")] + list(extra_flags or [])
    tmp = LIB + ".tmp%d" % os.getpid()
    objs = [f"{tmp}.{i}.o" for i in range(len(SOURCES))]
    cmds = [[hipcc(), *flags, "-c", src, "-o", obj] for src, obj in zip(SOURCES, objs)]
    link = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-o", tmp, *objs]
    if verbose:
        print("\n".join(" ".join(c) for c in cmds + [link]), flush=True)
    try:
        procs = [subprocess.Popen(c, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
                 for c in cmds]
        outs = [(p.communicate()[0], p.returncode) for p in procs]
        res = subprocess.run(link, capture_output=True, text=True) if all(
            rc == 0 for _, rc in outs) else None
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    text = "".join(t for t, _ in outs) + (res.stdout + res.stderr if res else "")
    if res is None or res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + text)
    if verbose and text:
        print(text, file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="--verbose" in sys.argv))

"""Build ``libsoma.so`` (the HIP library behind include/soma.h) for gfx950.

Run ``python -m paper_2609_37899_amd.build`` (or ``__graft_entry__.build()``).
The library is built in-tree next to this file.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRCS = [os.path.join(PKG, "csrc", f) for f in ("soma_api.hip", "soma_rec.hip")]
LIB = os.path.join(PKG, "libsoma.so")
ARCH = os.environ.get("SOMA_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++20", "-fPIC",
    # The probe generator is specified operation by operation: no contraction.
    "-ffp-contract=off",
    # Packed fp32 VALU instructions (v_pk_*_f32) stay off: plain fp32 code
    # is compiled to single-lane instructions only.
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # The instruction scheduler's ILP strategy: the body kernel runs one wave
    # per SIMD, so its latencies are hidden only by independent instructions
    # of the same wave (measured: 35.4 -> 27.2 ms per step on the body
    # workload, 113.4 -> 111.7 ms on the stacked-LSTM workload).
    "-mllvm", "-amdgpu-sched-strategy=max-ilp",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def build(verbose: bool = False) -> str:
    """Compile the translation units side by side, then link them."""
    tmp = LIB + ".tmp%d" % os.getpid()
    objs = [tmp + ".%d.o" % i for i in range(len(SRCS))]
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]
    cmds = [[hipcc(), *HIPCC_FLAGS, *inc, "-c", "-o", o, s] for s, o in zip(SRCS, objs)]
    try:
        for cmd in cmds if verbose else []:
            print(" ".join(cmd), flush=True)
        procs = [subprocess.Popen(cmd, cwd="/tmp") for cmd in cmds]
        codes = [p.wait() for p in procs]
        for code, cmd in zip(codes, cmds):
            if code:
                raise subprocess.CalledProcessError(code, cmd)
        subprocess.check_call([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs], cwd="/tmp")
    finally:
        for o in objs:
            if os.path.exists(o):
                os.unlink(o)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

"""Build the HIP library (liblbg.so) for gfx950, in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB_PATH = os.path.join(HERE, "liblbg.so")
SOURCES = [os.path.join(HERE, "csrc", "lbg.hip")]
DEPS = SOURCES + [os.path.join(HERE, "csrc", f) for f in ("lbg_device.hpp", "lbg_kernels.hpp", "lbg_sliced.hpp",
                                                                    "lbg_split.hpp", "lbg_order.hpp",
                                                                    "lbg_team.hpp", "lbg_pull.hpp", "lbg_solo.hpp",
                                                                    "lbg_sym.hpp")] + \
    [os.path.join(ROOT, "include", "lbg.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep the compiler from forming packed-FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    tmp = LIB_PATH + ".tmp"
    cmd = [hipcc(), *HIPCC_FLAGS, "-o", tmp, *SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))

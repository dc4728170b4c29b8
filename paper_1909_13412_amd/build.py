"""Build the HIP C-ABI library liblbmbp.so in-tree for gfx950 (hipcc cross-compiles
without a GPU)."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRCS = [os.path.join(PKG, "csrc", name) for name in (
    "lbmbp.hip", "twostep.hip", "collide_f64.hip", "collide_f32.hip", "collide_bf16.hip", "collide_f16.hip")]
LIB = os.path.join(PKG, "liblbmbp.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    # packed FP32 instructions stay off in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose: bool = False) -> str:
    """Compile every HIP source of the package into liblbmbp.so (always rebuilds;
    the translation units compile side by side)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]
    objs = [src + ".o" for src in SRCS]
    runs = [subprocess.Popen([hipcc, *HIPCC_FLAGS, *inc, "-c", "-o", obj, src], stdout=subprocess.PIPE,
                             stderr=subprocess.STDOUT, text=True) for src, obj in zip(SRCS, objs)]
    outs = [run.communicate()[0] for run in runs]
    for run, out in zip(runs, outs):
        if run.returncode != 0:
            raise RuntimeError(f"hipcc failed ({run.returncode}):\n{out}")
        if verbose and out:
            print(out)
    tmp = LIB + ".tmp"
    res = subprocess.run([hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs],
                         capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed ({res.returncode}):\n{res.stderr}")
    os.replace(tmp, LIB)
    for obj in objs:
        os.remove(obj)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

"""Build libzp.so (HIP kernels + C ABI) for gfx950 with hipcc, in tree."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libzp.so")
SOURCES = ["zp_mfma_d128_wide_ref.hip", "zp_mfma_d128_ref.hip", "zp_mfma_d64_wide_ref.hip", "zp_mfma_d128_wide.hip", "zp_mfma_d64_ref.hip",
           "zp_mfma_d128.hip", "zp_mfma_d64_wide.hip", "zp_mfma_d64.hip", "zp_mfma_pad_bf16.hip", "zp_mfma_pad_bf16_long.hip",
           "zp_mfma_pad_f32.hip", "zp_kernels.hip", "zp_check.hip", "zp_api.hip"]       # the slowest to compile first
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def build(verbose: bool = False) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)   # host pass does not know the feature
        if r.returncode:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), 8)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    # stand-alone counter/timing driver, linked against the library it measures
    drv = os.path.join(HERE, "zp_prof_driver")
    r = subprocess.run(["hipcc", *FLAGS, os.path.join(CSRC, "zp_prof_driver.hip"), "-o", drv, "-L" + HERE, "-lzp", "-Wl,-rpath,$ORIGIN"],
                       capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("driver build failed:\n" + r.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

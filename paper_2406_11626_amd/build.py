"""Builds the HIP library libccz4.so (gfx950) in this package directory."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libccz4.so")
SOURCES = ["ccz4_lds_fp64.hip", "ccz4_lds_fp64_lop.hip", "ccz4_lds_mixed.hip", "ccz4_lds_mixed_lop.hip",
           "ccz4_kernels.hip", "ccz4_mlp.hip", "ccz4_host.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unused-result"]


def build(verbose=False, out=OUT, defines=()):
    os.makedirs(os.path.join(CSRC, "_build"), exist_ok=True)
    tag = "".join(d.replace("=", "") for d in defines)

    def compile_one(src):
        obj = os.path.join(CSRC, "_build", tag + src + ".o")
        cmd = [HIPCC, "-x", "hip", *FLAGS, *["-D" + d for d in defines], "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1, 8)) as pool:
        objs = list(pool.map(compile_one, SOURCES))
    tmp = out + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

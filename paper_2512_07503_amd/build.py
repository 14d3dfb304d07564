"""Builds the HIP library (gfx950) into paper_2512_07503_amd/libsjd.so with hipcc."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsjd.so")
BUILD = os.path.join(HERE, "_build")

COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          # packed-fp32 code generation is switched off (hipcc's host pass warns that it does not know the feature)
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          # leading scalar arguments of a kernel arrive in registers instead of through a load
          "-mllvm", "-amdgpu-kernarg-preload-count=14"]
# (source, extra flags): the decision stage is specified bit for bit and must not contract a*b+c
UNITS = [("decide.hip", ["-ffp-contract=off"]), ("sjd_api.hip", [])]


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    objs = []
    for src, extra in UNITS:
        obj = os.path.join(BUILD, src.replace(".hip", ".o"))
        cmd = ["hipcc"] + COMMON + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if verbose and err.strip():
            print(err, flush=True)
        objs.append(obj)
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)

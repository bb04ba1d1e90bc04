"""Build the HIP library librmhdlb.so for gfx950 in-tree.

Every call compiles (the build check runs without a GPU: hipcc cross-compiles
gfx950).  Packed-FP32 instructions are disabled on every HIP translation unit.
"""
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "librmhdlb.so")
# (source, object, extra flags): the kernels compile once per storage form, side by side
UNITS = [("rmhdlb_api.hip", "rmhdlb_api.o", []), ("rmhdlb_mlp.hip", "rmhdlb_mlp.o", [])] + [
    ("rmhdlb_kernels.hip", f"rmhdlb_kernels_f{form}.o", [f"-DRMHDLB_FORM={form}"]) for form in (64, 32, 16)]
ARCH = os.environ.get("RMHDLB_ARCH", "gfx950")
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]


def hipcc():
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def build(verbose=False):
    objs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    procs = []
    for src, name, extra in UNITS:  # translation units compile in parallel
        obj = os.path.join(bdir, name)
        cmd = [hipcc()] + FLAGS + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)))
        objs.append(obj)
    failed = []
    for src, p in procs:
        _, err = p.communicate()
        if p.returncode != 0:
            sys.stderr.write(err)
            failed.append(src)
    if failed:
        raise RuntimeError(f"hipcc failed on {', '.join(failed)}")
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)

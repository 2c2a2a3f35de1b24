"""Build libtq.so (the HIP library behind include/tq.h) for gfx950 with hipcc, and _tqpy.so (the
native half of the Python binding) with g++, in-tree."""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(ROOT, "_build", "tq")
LIB = os.path.join(HERE, "libtq.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
# No fast-math: the activation quantizer relies on correctly rounded fp32 division and
# an unfused multiply. Packed-fp32 instructions are disabled on the device.
COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str, obj_dir: str = OBJ, defines=()) -> str:
    obj = os.path.join(obj_dir, os.path.basename(src) + ".o")
    cmd = [HIPCC, *COMMON, *[f"-D{d}" for d in defines], "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False, out: str = LIB, defines=(), obj_dir: str = OBJ) -> str:
    """Compile every source under csrc/ and link `out`. `defines` (NAME=VALUE strings)
    override build-time tile shapes."""
    os.makedirs(obj_dir, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, obj_dir, defines), srcs))
    tmp = out + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)
    if verbose:
        print(out)
    return out


def build_py() -> str:
    """Compile the native half of the Python binding (_tqpy.so) against the running torch."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    src, out = os.path.join(HERE, "csrc_py", "tq_py.cpp"), os.path.join(HERE, "_tqpy.so")
    inc = [f"-isystem{p}" for p in [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]]]
    libs = [f"-L{p}" for p in cpp_extension.library_paths()]
    tmp = out + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           *inc, src, "-o", tmp, *libs, "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for {src}:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)
    return out


def device_asm(src: str) -> str:
    """gfx950 assembly of one source file (for inspection)."""
    out = os.path.join(OBJ, os.path.basename(src) + ".s")
    os.makedirs(OBJ, exist_ok=True)
    cmd = [HIPCC, *COMMON, "--cuda-device-only", "-S", src, "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    return open(out).read()


if __name__ == "__main__":
    build(verbose=True)
    print(build_py())
    sys.exit(0)

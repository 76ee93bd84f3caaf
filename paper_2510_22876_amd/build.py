"""Build libspecdec.so for gfx950 with hipcc (in-tree, next to this file).

Usage: ``python -m paper_2510_22876_amd.build``.  Every HIP source is compiled
with packed-FP32 instructions disabled (``-packed-fp32-ops``).  The native
argument marshalling of the Python binding (``_marshal``, host code against
torch's headers) is built beside it, for the interpreter and the torch that
build it.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
CSRC = PKG / "csrc"
LIB = PKG / "libspecdec.so"
MARSHAL = PKG / ("_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
ARCH = "gfx950"

COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          f"-I{ROOT / 'include'}", f"-I{CSRC}"]


def build(verbose: bool = False, defines=(), out: Path = LIB, build_dir: Path | None = None) -> Path:
    """Compile every source under csrc/ and link ``out``.  ``defines`` adds
    -D options (the kernels' compile-time tunables)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    out_dir = build_dir or (PKG / "_build")
    out_dir.mkdir(parents=True, exist_ok=True)
    extra = [f"-D{d}" for d in defines]
    for src in sorted(CSRC.glob("*.hip")) + sorted(CSRC.glob("*.cpp")):
        obj = out_dir / (src.name + ".o")
        cmd = [hipcc, *COMMON, *extra, "-c", str(src), "-o", str(obj)]
        if src.suffix == ".cpp":
            cmd = [hipcc, *COMMON, *extra, "-x", "hip", "-c", str(src), "-o", str(obj)]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        objs.append(str(obj))
    tmp = Path(out).with_suffix(".so.tmp")
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", str(tmp)]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return Path(out)


def build_marshal(verbose: bool = False) -> Path | None:
    """Compile the extension module ``_marshal`` (host code only).  The binding
    does without it, so where the compiler or torch's and Python's headers are
    not there, what an earlier build left is removed and None is returned."""
    import torch
    root = Path(torch.__file__).resolve().parent
    cxx = os.environ.get("CXX", "g++")
    include = sysconfig.get_paths()["include"]
    needed = (root / "include" / "ATen" / "core" / "Tensor.h", Path(include) / "Python.h")
    if not shutil.which(cxx.split()[0]) or not all(h.exists() for h in needed):
        print(f"{MARSHAL.name} is not built: {cxx}, {needed[0]} and {needed[1]} are needed", file=sys.stderr, flush=True)
        MARSHAL.unlink(missing_ok=True)
        return None
    tmp = MARSHAL.with_suffix(".so.tmp")
    cmd = [*cxx.split(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DSPECDEC_TORCH_VERSION="{torch.__version__}"',
           f"-I{ROOT / 'include'}", f"-isystem{root / 'include'}", f"-I{include}",
           str(CSRC / "python" / "marshal.cpp"), f"-L{root / 'lib'}", "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-o", str(tmp)]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, MARSHAL)
    return MARSHAL


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    build_marshal(verbose="-v" in sys.argv)
    print(LIB)

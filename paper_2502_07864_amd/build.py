"""Build the gfx950 shared library in-tree with hipcc.

``python -m paper_2502_07864_amd.build`` compiles every ``csrc/*.hip`` for
gfx950 and links ``libmla_gfx950.so`` next to this file.  hipcc
cross-compiles, so this works on a machine without a GPU.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path
from typing import Optional

PKG = Path(__file__).resolve().parent
CSRC = PKG / "csrc"
INCLUDE = PKG.parent / "include"
OBJDIR = PKG / "_build"
LIB = PKG / "libmla_gfx950.so"
MARSHAL = PKG / ("_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Wall", "-Wno-unused-function",
    # never let the compiler form packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not Path(exe).exists():
        raise RuntimeError("hipcc not found (need ROCm to build the gfx950 library)")
    return exe


def sources():
    return sorted(CSRC.glob("*.hip"))


def build_marshal() -> Optional[Path]:
    """The Python extension that hands tensors to the library's entry points (host code only: g++, or the clang++ that
    comes with hipcc).  The library and its binding work without it, so where it cannot be built (no torch, no
    headers) this warns and leaves none behind: mla.py then passes every argument from Python."""
    MARSHAL.unlink(missing_ok=True)
    try:
        import torch
    except ImportError as e:
        warnings.warn(f"the marshalling extension is not built: {e}", RuntimeWarning)
        return None
    root = Path(torch.__file__).resolve().parent
    rocm = Path(hipcc()).resolve().parents[1]
    cxx = shutil.which("g++") or str(rocm / "llvm" / "bin" / "clang++")
    tmp = MARSHAL.with_suffix(".so.tmp")
    cmd = [cxx, "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f"-I{INCLUDE}", f"-I{sysconfig.get_paths()['include']}", f"-I{root / 'include'}",
           f"-I{root / 'include' / 'torch' / 'csrc' / 'api' / 'include'}", f"-I{rocm / 'include'}",
           str(CSRC / "marshal.cpp"), "-o", str(tmp), f"-L{root / 'lib'}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
    except OSError as e:
        warnings.warn(f"the marshalling extension is not built: {e}", RuntimeWarning)
        return None
    if r.returncode != 0:
        warnings.warn(f"the marshalling extension is not built: {cxx} failed on marshal.cpp:\n{r.stdout}{r.stderr}", RuntimeWarning)
        return None
    os.replace(tmp, MARSHAL)
    return MARSHAL


def build_library(verbose: bool = False, extra_flags=()) -> Path:
    OBJDIR.mkdir(exist_ok=True)
    cc = hipcc()

    def compile_one(src: Path) -> Path:
        obj = OBJDIR / (src.stem + ".o")
        cmd = [cc, *HIPCC_FLAGS, *extra_flags, "-c", str(src), "-o", str(obj)]
        r = subprocess.run(cmd, capture_output=True, text=True)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                        if "packed-fp32-ops" not in l and "target feature" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src.name}:\n{r.stdout}{r.stderr}")
        if verbose and out.strip():
            print(out)
        return obj

    def check_pending_registers() -> None:
        # decode_mfma.hip's query rows: loads with register outputs awaited later by count (asm_checks.py)
        from .asm_checks import check_listing
        src = CSRC / "decode_mfma.hip"
        asm = OBJDIR / "decode_mfma.s"
        cmd = [cc, *HIPCC_FLAGS, *extra_flags, "-S", "--cuda-device-only", str(src), "-o", str(asm)]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc -S failed on {src.name}:\n{r.stdout}{r.stderr}")
        seen = check_listing(asm.read_text(), "decode_mfma_kernel")
        if not seen or not all(seen.values()):
            raise RuntimeError(f"asm check found no query-row loads to look at in {sorted(seen)}")

    with ThreadPoolExecutor(max_workers=min(4, os.cpu_count() or 1)) as ex:
        check = ex.submit(check_pending_registers)
        marshal = ex.submit(build_marshal)
        objs = list(ex.map(compile_one, sources()))
        check.result()
        marshal.result()
    tmp = LIB.with_suffix(".so.tmp")
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", str(tmp), *map(str, objs)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))

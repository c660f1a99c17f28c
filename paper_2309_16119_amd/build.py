"""Build libmodulora.so (HIP, gfx950 only) and the host-side module _marshal.so in-tree with hipcc.

    python -m paper_2309_16119_amd.build          # compile every source, link

The shared object lands next to this file so that it travels with the source
tree; nothing is installed into site-packages and there is no JIT cache.
"""
from __future__ import annotations

import importlib.util
import os
import runpy
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libmodulora.so")
MARSHAL = os.path.join(PKG, "_marshal.so")

SOURCES = ["api.hip", "dequant_kernel.hip", "gemm_tile.hip", "gemm_big.hip", "gemm_big_192.hip", "gemm_mid.hip", "gemm_direct.hip", "finish.hip", "lora_kernels.hip", "smallm.hip", "single.hip", "optim.hip", "quantize.hip", "f16_path.hip", "bench_hooks.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-variable", "-Wno-unused-but-set-variable",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str, extra: list[str]) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, res.stdout, res.stderr))
    return obj


def _torch_dir() -> str | None:
    """Where torch is installed, if its headers and libraries for AMD GPUs are there too."""
    spec = importlib.util.find_spec("torch")
    root = os.path.dirname(spec.origin) if spec and spec.origin else None
    needed = (("include", "c10", "hip", "HIPStream.h"), ("lib", "libc10_hip.so"))
    return root if root and all(os.path.exists(os.path.join(root, *path)) for path in needed) else None


def _build_marshal() -> bool:
    """The module that hands tensors to the library: host code against torch's headers.  False without them: the
    library itself needs no torch, and binding.py does its calls without the module."""
    torch_dir = _torch_dir()
    if torch_dir is None:
        return False
    inc = [os.path.join(ROOT, "include"), "/opt/rocm/include", os.path.join(torch_dir, "include"),
           os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"]]
    libs = os.path.join(torch_dir, "lib")
    version = runpy.run_path(os.path.join(torch_dir, "version.py"))
    tmp = MARSHAL + ".tmp.%d" % os.getpid()
    cmd = [_hipcc(), "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           '-DMARSHAL_TORCH="%s %s"' % (version["__version__"], version["git_version"]), *("-I" + d for d in inc), os.path.join(CSRC, "marshal.cpp"), "-o", tmp, "-L" + libs, "-ltorch_python", "-ltorch", "-ltorch_cpu",
           "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for marshal.cpp:\n%s\n%s" % (res.stdout, res.stderr))
    os.replace(tmp, MARSHAL)
    return True


def build_library(extra_flags: list[str] | None = None, verbose: bool = False) -> str:
    """Compile every HIP source for gfx950, link the shared library and build the host module (where torch's headers are
    there; whatever becomes of it, the library is linked).  Always rebuilds."""
    os.makedirs(OBJ, exist_ok=True)
    extra = list(extra_flags or [])
    with ThreadPoolExecutor(max_workers=8) as ex:
        marshal = ex.submit(_build_marshal)
        objs = list(ex.map(lambda s: _compile(s, extra), SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (res.stdout, res.stderr))
    os.replace(tmp, LIB)
    if not marshal.result():
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)           # of another torch
        print("no torch headers for AMD GPUs: built without", os.path.basename(MARSHAL), file=sys.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_library(sys.argv[1:], verbose=True)

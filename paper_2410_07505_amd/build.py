"""Build libcrossquant.so (hand-written HIP for gfx950) in-tree with hipcc, and the binding's native part with g++.

    python -m paper_2410_07505_amd.build

Cross-compiles without a GPU.  The shared libraries are placed next to this file so that they
travel with the source tree.
"""
from __future__ import annotations

import importlib.machinery
import importlib.util
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libcrossquant.so")
SOURCES = ["cq_api.hip", "cq_slots.hip", "cq_absmax.hip", "cq_quantize.hip", "cq_analysis.hip", "cq_fused.hip", "cq_weight.hip", "cq_gemm.hip", "cq_gemm_staged.hip", "cq_gemm_wide.hip", "cq_gemm_fusedq.hip", "cq_gemm_fp6.hip", "cq_ceilings.hip"]

# The binding's own native part (no device code): built against the Python and torch that run this.
FASTCALL = os.path.join(HERE, "_fastcall" + importlib.machinery.EXTENSION_SUFFIXES[0])

# -ffp-contract=off: every binary32 operation rounds on its own (results are specified bit for
# bit).  -packed-fp32-ops off: packed FP32 VALU forms are not used on the test machines.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
               "-fno-fast-math", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def _torch_version(torch_dir: str) -> str:
    spec = importlib.util.spec_from_file_location("torch_version", os.path.join(torch_dir, "version.py"))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module.__version__


def _build_fastcall() -> None:
    if os.path.exists(FASTCALL):
        os.remove(FASTCALL)                   # none rather than one of another library's age
    found = importlib.util.find_spec("torch")
    if found is None:
        raise RuntimeError("no torch to build the binding's native part for")
    torch = found.submodule_search_locations[0]
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = FASTCALL + ".tmp%d" % os.getpid()
    includes = [os.path.join(torch, "include"), os.path.join(torch, "include", "torch", "csrc", "api", "include"),
                os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           '-DCQ_TORCH_VERSION="%s"' % _torch_version(torch),
           *("-I" + i for i in includes), os.path.join(CSRC, "cq_fastcall.cpp"), "-o", tmp,
           "-L" + os.path.join(torch, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed for cq_fastcall.cpp:\n" + res.stdout)
    os.replace(tmp, FASTCALL)


def build(extra_flags=(), verbose: bool = False) -> str:
    """The library; and the binding's native part, without which every call goes through the Python checks, where there is a
    torch with headers and a g++ to build it: where that fails, the library is built all the same and a line says so."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        fastcall = ex.submit(_build_fastcall)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stdout)
    os.replace(tmp, LIB)
    failure = fastcall.exception()
    if failure is not None:
        sys.stderr.write("the binding's native part is not built: %s\n" % failure)
    if verbose:
        print("built", LIB)
        if failure is None:
            print("built", FASTCALL)
    return LIB


if __name__ == "__main__":
    build(verbose=True)

"""Builds libsurel.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

``python -m paper_2202_13538_amd.build`` compiles every source under ``csrc/`` and links
``paper_2202_13538_amd/libsurel.so``, then the memory-system micro-benchmarks of
``membench/`` into ``libsurel_membench.so`` (benchmark tooling that ``bench.py --membench``
loads; the hot path does not), and ``_marshal.so``, the binding's argument checks, with the host
compiler.  Without a host compiler or torch's headers there is no ``_marshal.so``, and the binding checks
in Python.  hipcc cross-compiles for gfx950, so no GPU is needed to build.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libsurel.so")
MEMBENCH_SRC = os.path.join(PKG_DIR, "membench", "membench.hip")
MEMBENCH_LIB_PATH = os.path.join(PKG_DIR, "libsurel_membench.so")
MARSHAL_SRC = os.path.join(PKG_DIR, "host", "marshal.cpp")
MARSHAL_PATH = os.path.join(PKG_DIR, "_marshal.so")
BUILD_DIR = os.path.join(PKG_DIR, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
# Packed FP32 instructions are switched off for all device code of this library.
HIP_FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra",
             "-Wno-unused-parameter", "-Xclang", "-target-feature", "-Xclang",
             "-packed-fp32-ops"]


def sources() -> list[str]:
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str, extra: list[str]) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC, *HIP_FLAGS, *extra, "-c", src, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass does not know the packed-fp32 feature name; that warning is harmless
    noise = ("is not a recognized feature for this target", "1 warning generated",
             "warning generated when compiling for host")
    err = "\n".join(l for l in res.stderr.splitlines() if not any(n in l for n in noise))
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{res.stderr}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _link(objs: list[str], lib_path: str) -> None:
    tmp = lib_path + f".tmp{os.getpid()}"
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    os.replace(tmp, lib_path)


def _build_marshal() -> str | None:
    """The binding's argument checks, an extension module against the torch and Python that run this.
    Returns None, or why there is none (one of an earlier build is removed then)."""
    try:
        import sysconfig

        import torch
        from torch.utils import cpp_extension

        torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
        tmp = MARSHAL_PATH + f".tmp{os.getpid()}"
        cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
               f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
               f'-DSUREL_TORCH_VERSION="{torch.__version__}"',
               *(f"-isystem{path}" for path in cpp_extension.include_paths()),
               "-I" + sysconfig.get_paths()["include"], MARSHAL_SRC, "-o", tmp, "-L" + torch_lib,
               "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath," + torch_lib]
        res = subprocess.run(cmd, capture_output=True, text=True)
        why = None if res.returncode == 0 else f"{cmd[0]} failed on {MARSHAL_SRC}:\n{res.stderr}"
    except (ImportError, OSError) as e:
        why = str(e)
    if why is None:
        os.replace(tmp, MARSHAL_PATH)
    elif os.path.exists(MARSHAL_PATH):
        os.remove(MARSHAL_PATH)
    return why


def build(extra_flags: list[str] | None = None, verbose: bool = False) -> str:
    """Compile and link unconditionally.  Returns the path of libsurel.so."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    extra = list(extra_flags or [])
    srcs = sources()
    all_srcs = srcs + [MEMBENCH_SRC]
    wanted = {os.path.basename(s) + ".o" for s in all_srcs}
    for f in os.listdir(BUILD_DIR):           # objects of sources that no longer exist
        if f.endswith(".o") and f not in wanted:
            os.remove(os.path.join(BUILD_DIR, f))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(all_srcs))) as pool:
        marshal = pool.submit(_build_marshal)
        objs = list(pool.map(lambda s: _compile(s, extra), all_srcs))
        no_marshal = marshal.result()
    _link(objs[:-1], LIB_PATH)
    _link(objs[-1:], MEMBENCH_LIB_PATH)
    if no_marshal is not None:
        sys.stderr.write(f"{MARSHAL_PATH} is not built, the binding checks its arguments in Python: {no_marshal}\n")
    if verbose:
        print(f"built {LIB_PATH} from {len(srcs)} sources, {MEMBENCH_LIB_PATH}"
              + ("" if no_marshal is not None else f" and {MARSHAL_PATH}") + " from 1")
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)

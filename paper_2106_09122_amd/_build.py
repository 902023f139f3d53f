"""Compile the HIP sources of psflib into ``libpsflib.so`` (gfx950) and the
native part of the Python binding into ``_psfop.so``, in-tree.

Each translation unit is compiled to an object under ``_build/`` in
parallel, then linked into a shared library next to this file.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB_PATH = os.path.join(PKG_DIR, "libpsflib.so")
SOURCES = ["psflib.hip", "geometry.hip", "build.hip", "build_lds.hip", "apply.hip", "gemm.hip", "model.hip", "grouped.hip", "spline.hip", "flux.hip", "probe.hip"]
BINDING = os.path.join(CSRC, "binding.cpp")
BINDING_PATH = os.path.join(PKG_DIR, "_psfop.so")
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; ROCm is required to build psflib")


def compile_flags() -> list:
    return [
        f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall",
        "-I", INCLUDE, "-I", CSRC,
        # packed FP32 instructions are kept out of every kernel
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    ]


def binding_commands() -> list:
    """Commands that compile and link the native binding against libpsflib.so
    (found next to it at run time) and the installed torch."""
    import torch
    t = os.path.dirname(torch.__file__)
    obj = os.path.join(BUILD_DIR, "binding.o")
    cxx = shutil.which("g++") or "g++"
    return [
        [cxx, "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
         "-DTORCH_API_INCLUDE_EXTENSION_H", "-DTORCH_EXTENSION_NAME=_psfop", "-I", INCLUDE,
         "-isystem", os.path.join(t, "include"),
         "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
         "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
         "-c", BINDING, "-o", obj],
        [cxx, "-shared", "-fPIC", obj, "-o", BINDING_PATH + ".tmp", "-L", os.path.join(t, "lib"),
         "-ltorch", "-ltorch_cpu", "-ltorch_python", "-lc10", "-lc10_hip", "-L", PKG_DIR,
         "-l:" + os.path.basename(LIB_PATH), "-Wl,-rpath,$ORIGIN"],
    ]


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every source, link libpsflib.so and the native binding; returns
    the path of libpsflib.so."""
    cc = hipcc()
    os.makedirs(BUILD_DIR, exist_ok=True)
    flags = compile_flags()

    def one(src):
        obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
        cmd = [cc, *flags, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        if verbose and r.stderr.strip():
            print(r.stderr)
        return obj

    def run(cmd, what):
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"{what} failed:\n{r.stdout}\n{r.stderr}")

    # a failed build must not leave an older library looking current
    for path in (LIB_PATH, BINDING_PATH):
        if os.path.exists(path):
            os.remove(path)
    compile_binding, link_binding = binding_commands()
    with ThreadPoolExecutor(max_workers=max(1, min(jobs, len(SOURCES) + 1))) as ex:
        binding = ex.submit(run, compile_binding, "compiling the binding")
        objs = list(ex.map(one, SOURCES))
        binding.result()
    tmp = LIB_PATH + ".tmp"
    cmd = [cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    run(cmd, "link")
    os.replace(tmp, LIB_PATH)
    run(link_binding, "linking the binding")
    os.replace(BINDING_PATH + ".tmp", BINDING_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))

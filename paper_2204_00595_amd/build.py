"""Builds libmonarch.so (HIP, gfx950; no torch involved) in-tree with hipcc, then the binding's native module _native.so
(host code over torch's C++ API) with the C++ compiler."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmonarch.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["monarch_api.hip", "monarch_generic.hip", "monarch_mfma.hip", "monarch_mfma_fwd_wide.hip", "monarch_mfma_fwd_frag.hip", "monarch_mfma_fwd_split.hip", "monarch_mfma_tiled.hip", "monarch_project.hip", "monarch_complex.hip", "monarch_stage_mfma.hip", "monarch_act.hip", "monarch_ops.hip",
           "monarch_mfma_bwd_wide.hip", "monarch_mfma_bwd_split.hip", "monarch_mfma_y1.hip", "monarch_mfma_wgrad.hip", "monarch_mfma_sq64.hip", "monarch_mfma_sq16.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed-fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def _torch_dir() -> str:
    import torch
    return os.path.dirname(torch.__file__)


def compile_native(obj: str) -> subprocess.Popen:
    inc = os.path.join(_torch_dir(), "include")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-I" + inc, "-I" + os.path.join(inc, "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
           "-I/opt/rocm/include", "-c", os.path.join(CSRC, "monarch_torch.cpp"), "-o", obj]
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)


def link_native(obj: str) -> None:
    tmp = NATIVE + ".tmp%d" % os.getpid()
    subprocess.check_call([os.environ.get("CXX", "g++"), "-shared", "-o", tmp, obj, "-L" + os.path.join(_torch_dir(), "lib"),
                           "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-L" + HERE, "-l:libmonarch.so",
                           "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, NATIVE)


def build(verbose: bool = False, jobs: int = 4) -> str:
    """Compile every source to an object (in parallel) and link libmonarch.so."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    native_obj = os.path.join(objdir, "monarch_torch.o")
    native = compile_native(native_obj)
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            for _, p in procs:
                if p.poll() is None:
                    p.wait()
                    break
    failed = False
    for src, p in procs:
        out = p.communicate()[0].decode()
        lines = [ln for ln in out.splitlines() if "packed-fp32-ops" not in ln]
        if p.returncode != 0:
            failed = True
            sys.stderr.write("\n".join(lines) + "\n")
        elif verbose and lines:
            print("\n".join(lines))
    if failed:
        raise RuntimeError("hipcc failed")
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    said = native.communicate()[0].decode()
    if native.returncode != 0:
        sys.stderr.write(said)
        raise RuntimeError("the native module did not compile")
    link_native(native_obj)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

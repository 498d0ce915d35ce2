"""Builds libssmscan.so (HIP, gfx950 only) in-tree with hipcc: one object per source, compiled in
parallel, then one link.  Beside it _ssmbind.so, the native half of the Python binding (host code only, against
torch's C++ headers), which is linked to the library."""
from __future__ import annotations

import concurrent.futures
import importlib.util
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libssmscan.so")
BIND = os.path.join(HERE, "_ssmbind.so")
BIND_SOURCE = os.path.join(CSRC, "pybind.cpp")
SOURCES = ["products2.hip", "products3.hip", "params.hip", "block.hip", "narrow.hip", "scan.hip", "ssm_api.hip", "gemm.hip", "noalloc.hip"]
HEADERS = [os.path.join(CSRC, h) for h in ("ssm_internal.h", "fast_div.h", "store_rule.h", "gemm_common.h", "gemm_kernel.h", "gemm_packed.h", "pk_units.h", "pack.h", "lookback.h")] + \
          [os.path.join(os.path.dirname(HERE), "include", h) for h in ("ssm.h", "ssm_measure.h")]
# packed-fp32 instructions are switched off on purpose (target feature removed for device code)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _newest_header() -> float:
    return max(os.path.getmtime(h) for h in HEADERS)


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(BIND):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, s) for s in SOURCES] + HEADERS
    return any(os.path.getmtime(d) > t for d in deps) or any(os.path.getmtime(d) > os.path.getmtime(BIND)
                                                             for d in [BIND_SOURCE] + HEADERS)


def _compile(hipcc: str, src: str, obj: str, verbose: bool) -> None:
    cmd = [hipcc] + FLAGS + ["-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def _bind_command(out: str):
    """The host compiler's command for the native half of the binding (torch is located, not imported)."""
    torch_dir = os.path.dirname(importlib.util.find_spec("torch").origin)
    inc, lib = os.path.join(torch_dir, "include"), os.path.join(torch_dir, "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-w",
            "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I" + inc, "-I" + os.path.join(inc, "torch", "csrc", "api", "include"),
            "-I" + sysconfig.get_paths()["include"], "-I/opt/rocm/include", BIND_SOURCE, "-o", out,
            "-L" + HERE, "-lssmscan", "-L" + lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python",
            "-Wl,-rpath,$ORIGIN"]


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every HIP source and link them into one shared library.  Returns its path.
    force=False recompiles only the objects that are older than their source or any header."""
    if not force and not is_stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJDIR, exist_ok=True)
    hdr_t = _newest_header()
    jobs = []
    for s in SOURCES:
        src = os.path.join(CSRC, s)
        obj = os.path.join(OBJDIR, s + ".o")
        fresh = os.path.exists(obj) and os.path.getmtime(obj) >= max(os.path.getmtime(src), hdr_t)
        if force or not fresh:
            jobs.append((src, obj))
    workers = max(1, min(len(jobs), len(os.sched_getaffinity(0)), 8))
    if jobs:
        with concurrent.futures.ThreadPoolExecutor(max_workers=workers) as pool:
            for f in [pool.submit(_compile, hipcc, src, obj, verbose) for src, obj in jobs]:
                f.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + [os.path.join(OBJDIR, s + ".o") for s in SOURCES] + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    if force or not os.path.exists(BIND) or os.path.getmtime(BIND) < max(os.path.getmtime(BIND_SOURCE), hdr_t):
        tmp = BIND + ".tmp%d" % os.getpid()
        cmd = _bind_command(tmp)
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        os.replace(tmp, BIND)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(force="--incremental" not in sys.argv, verbose=True))

"""Build libtri.so in-tree: gfx950 kernels with hipcc, the host cache core
with the system C++ compiler, linked against the HIP runtime.

`build()` always recompiles everything (a few tens of seconds on 8 cores).
`build_host_core(backend_src, out)` links the same host sources against
another launch backend (the CPU tests use a recording one).
"""
from __future__ import annotations

import concurrent.futures as cf
import importlib.util
import os
import re
import shutil
import subprocess
import sys
import sysconfig
from typing import List, Optional

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
KDIR = os.path.join(CSRC, "kernels")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libtri.so")
FAST_LIB = os.path.join(PKG, "_fast.so")
BENCH_LIB = os.path.join(PKG, "libtri_bench.so")
HOSTCOST_LIB = os.path.join(PKG, "libtri_hostcost.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.path.join(ROCM, "bin", "hipcc")
CXX = os.environ.get("CXX", "g++")

ARCH = "gfx950"
# Packed-FP32 instructions are disabled: hipcc may form v_pk_{add,mul,fma}_f32
# from ordinary float code, and we keep every float32 operation scalar.
# Floating-point contraction is off: a * b + c is never fused unless the
# source says fmaf, so a kernel's rounding steps do not depend on how the
# compiler schedules the surrounding code -- the precompiled kernels and a
# runtime-compiled specialization of the same body (which folds shape
# constants and unrolls differently) round identically.
DEVICE_FLAGS = ["-O3", "-std=c++17", "-ffp-contract=off",
                "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
HIP_FLAGS = [f"--offload-arch={ARCH}", *DEVICE_FLAGS, "-fPIC", "-I", INCLUDE, "-I", CSRC]
HOST_FLAGS = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra", "-I", INCLUDE, "-I", CSRC]
HOST_SOURCES = ["api.cpp", "cache.cpp", "policy.cpp", "jit.cpp", "tune.cpp", "resident.cpp"]
JIT_PRELUDE = os.path.join(BUILD, "jit_prelude.cpp")
HIP_BACKEND = "backend_hip.cpp"


def _run(cmd: List[str]) -> None:
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass warns that it does not know the packed-fp32 feature
    out = "\n".join(l for l in r.stdout.splitlines()
                    if "packed-fp32-ops' is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"command failed ({r.returncode}): {' '.join(cmd)}\n{out}")
    if out.strip():
        print(out, file=sys.stderr)


def write_jit_prelude(path: str = JIT_PRELUDE) -> str:
    """The device prelude of runtime-compiled specializations: kernargs.h and
    kernels/device.h as one text (their HIP-runtime and relative includes
    dropped; the runtime compiler provides the HIP device environment),
    embedded in the library as a C++ string constant."""
    text = []
    for rel in ("kernargs.h", os.path.join("kernels", "device.h")):
        with open(os.path.join(CSRC, rel)) as f:
            for line in f:
                if (line.startswith("#include <hip/") or line.startswith('#include "../kernargs.h"')
                        or line.startswith("#pragma once")):
                    continue
                text.append(line)
    body = "".join(text)
    delim = "TRIJIT"
    assert f"){delim}\"" not in body
    os.makedirs(os.path.dirname(path), exist_ok=True)
    src = ("// Generated by build.py from kernargs.h and kernels/device.h. Do not edit.\n"
           "#include <stdint.h>\n"
           "namespace tri {\n"
           f"extern const char kJitPrelude[] = R\"{delim}({body}){delim}\";\n"
           "extern const uint64_t kJitPreludeLen = sizeof(kJitPrelude) - 1;\n"
           "}  // namespace tri\n")
    old = open(path).read() if os.path.exists(path) else None
    if old != src:
        with open(path, "w") as f:
            f.write(src)
    return path


def _obj(src: str) -> str:
    return os.path.join(BUILD, os.path.basename(src) + ".o")


def torch_dir() -> Optional[str]:
    """The installed torch package's folder, found without importing it; None
    without torch."""
    spec = importlib.util.find_spec("torch")
    return spec.submodule_search_locations[0] if spec else None


def fast_compile_cmd(torch: str) -> List[str]:
    """The binding's native op calls (csrc/binding/fast.cpp) against the
    headers of the torch in folder `torch` and Python's."""
    inc = os.path.join(torch, "include")
    with open(os.path.join(torch, "version.py")) as f:
        version = re.search(r"__version__ = '([^']+)'", f.read()).group(1)
    src = os.path.join(CSRC, "binding", "fast.cpp")
    system = [inc, os.path.join(inc, "torch", "csrc", "api", "include"),
              os.path.join(ROCM, "include"), sysconfig.get_paths()["include"]]
    flags = [f for d in system for f in ("-isystem", d)]
    return [CXX, *HOST_FLAGS, "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
            f'-DTRI_TORCH_VERSION="{version}"', *flags, "-c", src, "-o", _obj(src)]


def hip_sources() -> List[str]:
    return sorted(os.path.join(KDIR, f) for f in os.listdir(KDIR) if f.endswith(".hip"))


def build(jobs: Optional[int] = None) -> str:
    """Compile and link libtri.so; returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(16, os.cpu_count() or 4)
    cmds = []
    for src in hip_sources():
        cmds.append([HIPCC, *HIP_FLAGS, "-c", src, "-o", _obj(src)])
    for name in HOST_SOURCES:
        src = os.path.join(CSRC, name)
        cmds.append([CXX, *HOST_FLAGS, "-c", src, "-o", _obj(src)])
    write_jit_prelude()
    cmds.append([CXX, *HOST_FLAGS, "-c", JIT_PRELUDE, "-o", _obj(JIT_PRELUDE)])
    src = os.path.join(CSRC, HIP_BACKEND)
    cmds.append([CXX, *HOST_FLAGS, "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                 "-c", src, "-o", _obj(src)])
    torch = torch_dir()
    fast = fast_compile_cmd(torch) if torch else None
    with cf.ThreadPoolExecutor(jobs) as ex:
        compiled = ex.submit(_run, fast) if fast else None
        for f in [ex.submit(_run, c) for c in cmds]:
            f.result()
    objs = [c[-1] for c in cmds]
    rocm_lib = os.path.join(ROCM, "lib")
    tmp = LIB + ".tmp"
    _run([CXX, "-shared", "-o", tmp, *objs, "-L", rocm_lib, "-lamdhip64", "-lhiprtc",
          "-Wl,-soname,libtri.so", f"-Wl,-rpath,{rocm_lib}", "-Wl,--no-undefined"])
    shutil.move(tmp, LIB)
    # the binding's extension module: libtri.so beside it, torch's libraries
    # as the process has loaded them; libtri.so needs neither and is there by now
    if fast:
        compiled.result()
        tmp = FAST_LIB + ".tmp"
        _run([CXX, "-shared", "-o", tmp, fast[-1], "-L", PKG, "-ltri", "-L",
              os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
              "-Wl,-rpath,$ORIGIN"])
        shutil.move(tmp, FAST_LIB)
    else:
        print("torch is not installed: libtri.so without the Python binding's extension module")
    # the benchmark's native timing loops, linked against libtri.so
    # and a reference streaming copy (the practical HBM ceiling)
    harness = os.path.join(CSRC, "bench", "harness.cpp")
    copy_src = os.path.join(CSRC, "bench", "copy.hip")
    _run([HIPCC, *HIP_FLAGS, "-c", copy_src, "-o", _obj(copy_src)])
    tmp = BENCH_LIB + ".tmp"
    _run([CXX, *HOST_FLAGS, "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
          "-shared", "-o", tmp, harness, _obj(copy_src), "-L", PKG, "-ltri", "-L", rocm_lib,
          "-lamdhip64", "-Wl,-rpath,$ORIGIN", f"-Wl,-rpath,{rocm_lib}", "-Wl,--no-undefined"])
    shutil.move(tmp, BENCH_LIB)
    # the host-cost microbenchmark: the cache core over a backend that
    # launches nothing (CPU only)
    bench_dir = os.path.join(CSRC, "bench")
    srcs = ([os.path.join(bench_dir, "hostcost.cpp"), os.path.join(bench_dir, "null_backend.cpp")]
            + [os.path.join(CSRC, n) for n in HOST_SOURCES if n != "api.cpp"] + [JIT_PRELUDE])
    tmp = HOSTCOST_LIB + ".tmp"
    _run([CXX, *HOST_FLAGS, "-shared", "-o", tmp, *srcs])
    shutil.move(tmp, HOSTCOST_LIB)
    return LIB


def build_host_core(backend_src: str, out: str, extra_flags: Optional[List[str]] = None) -> str:
    """Link the host cache core with `backend_src` into shared library `out`."""
    srcs = ([os.path.join(CSRC, n) for n in HOST_SOURCES] + [write_jit_prelude()]
            + [backend_src])
    tmp = out + ".tmp"
    _run([CXX, *HOST_FLAGS, *(extra_flags or []), "-shared", "-o", tmp, *srcs])
    shutil.move(tmp, out)
    return out


if __name__ == "__main__":
    print(build())

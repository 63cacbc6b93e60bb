"""Compile the HIP sources under csrc/ for gfx950 into csrc/libfptq.so, the measurement aids into csrc/libfptq_probe.so and
the Python binding's native fast path into _native.so (in-tree, so that the built libraries travel with the source tree)."""
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(CSRC, "libfptq.so")
PROBE_LIB = os.path.join(CSRC, "libfptq_probe.so")
SOURCES = ["fptq_api.hip", "fptq_pack.hip", "fptq_quant.hip", "fptq_gemm.hip", "fptq_prefill.hip", "fptq_gemv.hip", "fptq_hadamard.hip", "fptq_residual.hip"]
PROBE_SOURCES = ["fptq_probe.hip"]
NATIVE_SOURCE, NATIVE = "fptq_native.cpp", os.path.join(HERE, "_native.so")      # the binding's fast path: host code, torch's C++ API

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# The first 14 words of a kernel's arguments arrive in scalar registers with the dispatch, so a wave's first loads do not wait for a load of
# their addresses (firmware without it enters at a prologue that loads them).  What bounds the short launches is latency: 333 x 32003 x 2504
# 28.2 -> 27.8 us, Hadamard and RMS quantizers of 4096 rows 40.6 -> 40.0, a decode block 41.2 -> 41.0; large products as before.  The dispatch
# itself takes about 0.1 us longer, which shows where a launch is hardly more than that: up to 4 rows of 4096 values, scale given, 1.97 -> 2.08.
KERNARG_PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         *KERNARG_PRELOAD,
         "-Wall", "-Wno-unused-command-line-argument", "-I", INCLUDE, "-I", CSRC]


def _compile(src):
    obj = os.path.join(CSRC, src.replace(".hip", ".o"))
    p = subprocess.run([HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode:
        raise RuntimeError(f"hipcc failed on {src}:\n{out}")
    return obj, out


def _native_command(obj):
    import torch
    from torch.utils import cpp_extension
    inc = ["-I", INCLUDE] + [f for d in [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]] for f in ("-isystem", d)]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-Wextra", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc,
            "-c", os.path.join(CSRC, NATIVE_SOURCE), "-o", obj]


def _link_native(obj):
    from torch.utils import cpp_extension
    dirs = [f"-L{d}" for d in cpp_extension.library_paths()]
    subprocess.check_call(["g++", "-shared", obj, "-o", NATIVE, *dirs, "-ltorch_python", "-ltorch_cpu", "-lc10", f"-L{CSRC}", "-l:libfptq.so",
                           "-Wl,-rpath,$ORIGIN/csrc"])


def build(verbose: bool = False) -> str:
    native_obj = os.path.join(CSRC, "fptq_native.o")
    with ThreadPoolExecutor(max_workers=len(SOURCES) + len(PROBE_SOURCES) + 1) as ex:
        native = ex.submit(subprocess.run, _native_command(native_obj), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        results = list(ex.map(_compile, SOURCES + PROBE_SOURCES))
    if verbose:
        for _, out in [*results, ("", native.result().stdout)]:
            if out.strip():
                print(out)
    objs = [o for o, _ in results]
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs[:len(SOURCES)], "-o", LIB])
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs[len(SOURCES):], "-o", PROBE_LIB])
    if native.result().returncode:
        raise RuntimeError(f"g++ failed on {NATIVE_SOURCE}:\n{native.result().stdout}")
    _link_native(native_obj)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

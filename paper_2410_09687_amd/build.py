"""Builds libmoin.so (gfx950 only) in-tree with hipcc, and the native half of moin.py against it.

``python -m paper_2410_09687_amd.build`` or ``build_libmoin()``.  Objects go to
``_build/`` (not tracked); the shared library lands next to this file so that
it travels with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libmoin.so")
BINDING = os.path.join(HERE, "_moin_binding.so")
SOURCES = ["api.hip", "plan.hip", "linear.hip", "linear_stream.hip", "linear_mid.hip", "decode.hip", "route.hip", "route_exact.hip", "kmeans.hip", "cache.hip", "mx.hip", "probe.hip", "merge.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _start_binding():
    """Compiles csrc/binding.cpp (host code; it needs torch's headers), beside the kernels."""
    import sysconfig

    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    obj = os.path.join(HERE, "_build", "binding.o")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-Wall", "-I" + inc,
           "-I" + sysconfig.get_paths()["include"], f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj]
    return obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _link_binding(obj):
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = BINDING + ".tmp"
    r = subprocess.run([os.environ.get("CXX", "g++"), "-shared", obj, "-o", tmp, "-L" + lib, "-ltorch_python", "-ltorch_cpu",
                        "-lc10", "-L" + HERE, "-l:libmoin.so", "-Wl,-rpath,$ORIGIN"], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link of the binding failed:\n" + r.stderr)
    os.replace(tmp, BINDING)


def build_libmoin(verbose: bool = False) -> str:
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(bdir, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass does not know the packed-fp32 feature switch and says so: harmless
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    binding_obj, binding = _start_binding()
    with ThreadPoolExecutor(max_workers=min(len(SOURCES), 8)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = OUT + ".tmp"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, OUT)
    said, _ = binding.communicate()
    if binding.returncode != 0:
        raise RuntimeError("g++ failed on binding.cpp:\n" + said)
    _link_binding(binding_obj)
    return OUT


if __name__ == "__main__":
    print(build_libmoin(verbose=True))

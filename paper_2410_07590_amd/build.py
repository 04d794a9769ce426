"""Build libturborag_hip.so (gfx950, hipcc) and _tr_host.so (the binding's extension module, host compiler) in-tree.
`python -m paper_2410_07590_amd.build`."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libturborag_hip.so")
HOST = os.path.join(HERE, "_tr_host.so")
SOURCES = ["tr_api.hip", "tr_copy.hip", "tr_attn.hip", "tr_attn_f32.hip", "tr_linear.hip", "tr_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # packed fp32 VALU forms are kept off for every HIP translation unit
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str, extra) -> str:
    obj = os.path.join(CSRC, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_host() -> None:
    import sysconfig

    import numpy
    import torch
    from torch.utils import cpp_extension as ext
    include = ext.include_paths() + [sysconfig.get_paths()["include"], numpy.get_include()]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
    for d in include:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "py_host.cpp"), "-o", HOST]
    cmd += ["-L" + d for d in ext.library_paths()] + ["-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("the host compiler failed for py_host.cpp:\n%s" % res.stderr)
    if res.stderr.strip():
        sys.stderr.write(res.stderr)


def build(extra_flags=()) -> str:
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        host = ex.submit(_build_host)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
        host.result()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    return LIB


def needs_build() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(HOST):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(HOST))
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".h", ".cpp"))]
    deps.append(os.path.join(HERE, "..", "include", "turborag.h"))
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    print(build(sys.argv[1:]))

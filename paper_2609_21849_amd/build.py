"""Build libqgemm.so (HIP, gfx950) and the torch binding in-tree.

    python -m paper_2609_21849_amd.build

Each .hip file is compiled to an object in parallel, then linked into
paper_2609_21849_amd/libqgemm.so next to this file; csrc/torch_binding.cpp
(host code only) becomes _qgemm_torch.so beside it, linked against it. Without
g++ or torch only the library is built, which the package can do with.
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libqgemm.so")
BINDING = os.path.join(HERE, "_qgemm_torch.so")
ARCH = "gfx950"

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
COMMON = [
    "--offload-arch=" + ARCH, "-O3", "-std=c++20", "-fPIC",
    # packed-fp32 VALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep fp32 denormals (quantizer parity relies on IEEE behaviour)
    "-fno-gpu-flush-denormals-to-zero",
    "-I" + INCLUDE, "-I" + CSRC,
]


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def binding_lacks() -> str | None:
    """What is missing here to build the torch binding, or None."""
    if shutil.which("g++") is None:
        return "no g++"
    try:
        import torch  # noqa: F401
    except ImportError as e:
        return "no torch (%s)" % e
    return None


def _compile_binding() -> str:
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(HIPCC)))
    obj = os.path.join(BUILD_DIR, "torch_binding.o")
    cmd = [shutil.which("g++"), "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I" + INCLUDE, "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include"),
           "-isystem", "/opt/rocm/include", "-c", os.path.join(CSRC, "torch_binding.cpp"), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for torch_binding.cpp:\n%s" % r.stderr)
    return obj


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC, *COMMON, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stderr))
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max(1, min(len(srcs), os.cpu_count() or 1))) as ex:
        lacks = binding_lacks()
        binding = None if lacks else ex.submit(_compile_binding)
        objs = list(ex.map(_compile, srcs))
        binding_obj = binding.result() if binding else None
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s" % r.stderr)
    os.replace(tmp, LIB)
    if binding_obj is None:
        if os.path.exists(BINDING):
            os.remove(BINDING)  # of another build
        print("torch binding not built: %s" % lacks, file=sys.stderr)
    else:
        _link_binding(binding_obj)
    if verbose:
        print("built", LIB)
    return LIB


def _link_binding(binding_obj: str) -> None:
    import torch
    tl = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = BINDING + ".tmp%d" % os.getpid()
    cmd = [shutil.which("g++"), "-shared", "-o", tmp, binding_obj, "-L" + HERE, "-l:libqgemm.so",
           "-Wl,-rpath,$ORIGIN", "-L" + tl, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link of the torch binding failed:\n%s" % r.stderr)
    os.replace(tmp, BINDING)


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)

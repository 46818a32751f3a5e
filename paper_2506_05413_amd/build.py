"""Builds libsmoothrot.so (HIP, gfx950 only) with hipcc and _marshal (the binding's native half) with g++, in-tree.

_marshal is an extension module for the Python and the torch that run the build; its file name carries the Python ABI, and it
holds the torch version it was compiled against.

    python -m paper_2506_05413_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libsmoothrot.so")
MARSHAL = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["sr_api.hip", "fwht_quant.hip", "fwht_two_pass.hip", "fold_search.hip", "calib_fold.hip", "gemm_prefill.hip", "gemm_packed_stream.hip", "gemm_f6.hip", "gemm_f6_stream.hip", "gemm_decode.hip", "kv_quant.hip", "linear_decode.hip", "ceilings.hip"]

# packed-fp32 instructions are switched off on purpose (device code only)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _check_asm_loads() -> None:
    """The staged rotation kernels load rows with inline-assembly loads whose destination registers must not be
    touched before the matching wait (csrc/check_asm_loads.py): verified on the device assembly of this build."""
    asm = os.path.join(OBJ, "fwht_quant.s")
    dev_flags = [f for f in FLAGS if f not in ("-fPIC", "-fvisibility=hidden")]
    r = subprocess.run([_hipcc(), *dev_flags, "-S", "--cuda-device-only", os.path.join(CSRC, "fwht_quant.hip"), "-o", asm],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc -S failed for fwht_quant.hip:\n" + r.stderr[-2000:])
    r = subprocess.run([sys.executable, os.path.join(CSRC, "check_asm_loads.py"), asm], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("inline-assembly load check failed:\n" + r.stdout + r.stderr)


def _compile_marshal() -> str:
    """csrc/marshal.cpp -> object file: host code against the headers of the installed torch and Python."""
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(OBJ, "marshal.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DSR_TORCH_VERSION="%s"' % torch.__version__]
    cmd += [f for d in ("include", "include/torch/csrc/api/include") for f in ("-isystem", os.path.join(root, d))]
    cmd += ["-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"]]
    r = subprocess.run(cmd + ["-c", os.path.join(CSRC, "marshal.cpp"), "-o", obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for marshal.cpp:\n" + r.stderr)
    return obj


def _link_marshal(obj: str) -> None:
    """_marshal; torch's libraries are in the process when it is imported, libsmoothrot.so lies beside it."""
    import torch
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-shared", "-o", MARSHAL, obj, "-L", PKG, "-lsmoothrot", "-L", libs, "-ltorch_python", "-ltorch_hip", "-ltorch_cpu",
           "-lc10_hip", "-lc10", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link of _marshal failed:\n" + r.stderr)


def build(verbose: bool = True) -> str:
    """Compile every source and link both shared libraries; returns the path of libsmoothrot.so (linked first: it needs neither
    torch nor Python)."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        marshal = ex.submit(_compile_marshal)
        check = ex.submit(_check_asm_loads)
        objs = list(ex.map(_compile, SOURCES))
        check.result()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    _link_marshal(marshal.result())
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()

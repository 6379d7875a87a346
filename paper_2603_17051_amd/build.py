"""Build the HIP library (gfx950) in-tree, paper_2603_17051_amd/libastro.so, and beside it the CPython module of the binding."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libastro.so")
# (tagged with the Python it is built for: another one looks for another file)
NATIVE_PATH = os.path.join(PKG_DIR, "_binding_native" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ["astro_api.hip", "rope_scatter.hip", "attn_f32.hip", "attn_fwd_bf16.hip", "attn_bwd_bf16.hip", "profile.hip", "calib.hip", "nft_loss.hip"]
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wno-unused-value",
    # IEEE semantics for infinities are kept (no -ffinite-math-only): the forward's softmax
    # notices a reference that is too low by a row sum that overflows to +inf, and lanes that own
    # no key may hold inf / NaN that is never stored
    # packed fp32 VALU ops are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: the HIP library cannot be built")
    return exe


def build_library(verbose: bool = False) -> str:
    hipcc = _hipcc()
    obj_dir = os.path.join(PKG_DIR, "_build")
    os.makedirs(obj_dir, exist_ok=True)

    def compile_one(src: str) -> str:
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [hipcc, *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
        if verbose:
            sys.stderr.write(r.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB_PATH + ".tmp"
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


def build_native() -> str:
    """Host code only, against the installed torch's headers and libraries."""
    import torch  # where its headers are
    root = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(_hipcc())))
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        raise RuntimeError("no C++ compiler: the binding's module cannot be built")
    tmp = NATIVE_PATH + ".tmp"
    cmd = [cxx, "-std=c++17", "-O2", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DBUILT_FOR_TORCH="{torch.__version__} {torch.version.git_version}"',
           "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(rocm, "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "binding_native.cpp"), "-o", tmp,
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"building the binding's module failed:\n{r.stderr}")
    os.replace(tmp, NATIVE_PATH)
    return NATIVE_PATH


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
    print(build_native())

"""Build libtfx.so (HIP kernels + C ABI) for gfx950 with hipcc, and _call.so (the Python entry points' host path,
against the installed PyTorch's C++ headers) with g++, in-tree.

Usage: python -m paper_1901_05350_amd.build [--force]
"""
import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtfx.so")
CALL = os.path.join(HERE, "_call.so")
SOURCES = ["api.hip", "gemm.hip", "pointwise.hip", "conv.hip", "depthwise.hip", "tail.hip", "elementwise.hip", "gemm_f16.hip", "gemm_deep.hip", "gemm_direct.hip", "gemm_thin.hip", "conv_f16.hip", "pointwise_f16.hip", "pointwise_slab_f16.hip", "conv_gemm_f16.hip", "conv_stream_f16.hip", "chain.hip", "block.hip", "block_stream.hip", "block_tile.hip", "block_stream_f16.hip", "block_tile_f16.hip", "block_patch.hip", "block_patch_f16.hip", "block_rows_f16.hip", "block_rows.hip", "conv_window.hip"]
HEADERS = [os.path.join(CSRC, "tfx_internal.h"), os.path.join(CSRC, "stream_f16.h"), os.path.join(CSRC, "ragged.h"), os.path.join(CSRC, "split.h"), os.path.join(CSRC, "pair.h"), os.path.join(CSRC, "pack.h"), os.path.join(CSRC, "kernel_cost.h"), os.path.join(HERE, "..", "include", "tfx.h")]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-function",
         # packed fp32 VALU ops are kept off on this target
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the first 14 dwords of a kernel's plain arguments come in scalar registers instead of through memory, .3 - .5 us of a launch
         "-mllvm", "-amdgpu-kernarg-preload-count=16"]


def _hipcc():
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src, force):
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    path = os.path.join(CSRC, src)
    if force or _stale(obj, [path] + HEADERS):
        subprocess.run([_hipcc()] + FLAGS + ["-c", path, "-o", obj], check=True)
    return obj


def _compile_call(force):
    """The extension module links against libtfx.so beside it and torch's libraries, which `import torch` has loaded
    by the time the module is imported.  Without a host compiler there is none (the binding then does without)."""
    src = os.path.join(CSRC, "call.cpp")
    if not force and not _stale(CALL, [src, LIB] + HEADERS):
        return
    if shutil.which(os.environ.get("CXX", "g++")) is None:
        print("no host compiler: _call.so is not built")
        return
    import sysconfig
    import torch
    base = os.path.dirname(torch.__file__)
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
                    "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                    "-isystem", os.path.join(base, "include"), "-isystem", os.path.join(base, "include/torch/csrc/api/include"),
                    "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"], src, "-o", CALL,
                    "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10_hip", "-lc10",
                    "-L" + HERE, "-ltfx", "-Wl,-rpath,$ORIGIN"], check=True)


def build(force=False, verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, force), SOURCES))
    if force or _stale(LIB, objs):
        subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, check=True)
    _compile_call(force)
    if verbose:
        print("built", LIB, CALL)
    return LIB


if __name__ == "__main__":
    build(force="--force" in sys.argv, verbose=True)

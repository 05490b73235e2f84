"""Build libbnn.so (hand-written HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import platform
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from typing import Optional, Sequence

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbnn.so")
FASTCALL = os.path.join(HERE, "_fastcall.so")
TENSORCALL = os.path.join(HERE, "_tensorcall.so")
OBJ_DIR = os.path.join(HERE, "_build")
SOURCES = ["api.hip", "encode.hip", "im2col.hip", "gemm.hip", "gemm_lowk.hip", "gemm_fewrows.hip", "gemm_fp4.hip", "gemm_fp4_split.hip", "conv.hip", "conv_first_sign.hip", "conv_chain.hip", "conv_pointwise.hip", "conv_word.hip", "glue.hip", "mfma.hip", "control.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Packed-FP32 VALU forms are disabled for all device code of this library.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wall", "-Wno-unused-function",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]

# conv.hip, conv_first_sign.hip: the matrix-core first layer reads its accumulators on the vector unit; keeping them in
# ordinary vector registers (not accumulation registers) saves a move per element, and those
# moves queue behind the matrix instruction in flight.
EXTRA_FLAGS = {f: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] for f in ("conv.hip", "conv_first_sign.hip")}


# Checker build of the HOST side (argument validation, dispatch, launch code) with AddressSanitizer
# and UndefinedBehaviorSanitizer; device code is compiled as usual.  CPU-only use:
#   python paper_1911_04477_amd/build.py --sanitize
#   LD_PRELOAD="$(gcc -print-file-name=libasan.so) $(gcc -print-file-name=libubsan.so)" ASAN_OPTIONS=detect_leaks=0 \
#       BNN_SANITIZE=1 python -m pytest tests/test_abi_host.py
SAN_LIB = os.path.join(HERE, "libbnn_san.so")
SAN_FASTCALL = os.path.join(HERE, "_fastcall_san.so")
SAN_TENSORCALL = os.path.join(HERE, "_tensorcall_san.so")
# The run ends at the first finding.  Enums are left out: a C caller may hand over any int, and the library says so; so are the types of
# called functions (kernels picked by an expression), which gcc's runtime, preloaded above, does not know.
SAN_HOST_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host",
                  "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-sanitize=enum", "-Xarch_host",
                  "-fno-sanitize=function", "-Xarch_host",
                  "-fno-omit-frame-pointer", "-g"]


def build_sanitized() -> str:
    out_dir = os.path.join(OBJ_DIR, "san")
    os.makedirs(out_dir, exist_ok=True)
    flags = [f if f != "-O3" else "-O1" for f in FLAGS]

    def comp(src: str) -> str:
        obj = os.path.join(out_dir, os.path.splitext(src)[0] + ".o")
        subprocess.check_call([HIPCC, *flags, *SAN_HOST_FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src),
                               "-o", obj])
        return obj

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(comp, SOURCES))
    tmp = SAN_LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Xarch_host", "-fsanitize=address",
                           "-Xarch_host", "-fsanitize=undefined", *objs, "-o", tmp])
    os.replace(tmp, SAN_LIB)
    checks = ("-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined")
    build_fastcall(SAN_FASTCALL, checks)
    build_tensorcall(SAN_TENSORCALL, (*checks, "-fno-sanitize=vptr"))  # torch's types are not all there to compare with
    return SAN_LIB


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    subprocess.check_call([HIPCC, *FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj])
    return obj


def build_fastcall(out: str = FASTCALL, flags: Sequence[str] = ("-O2",)) -> Optional[str]:
    """The binding's call helper, a CPython extension.  None where it cannot be built (no Python headers, not x86-64): the
    binding then calls through ctypes."""
    if os.path.exists(out):
        os.remove(out)  # not one of another source
    include = sysconfig.get_paths()["include"]
    if platform.machine() != "x86_64" or not os.path.exists(os.path.join(include, "Python.h")):
        print("call helper not built: it needs x86-64 and", os.path.join(include, "Python.h"))
        return None
    cc = [shutil.which("gcc")] if shutil.which("gcc") else [HIPCC, "-x", "c"]
    tmp = out + ".tmp.%d" % os.getpid()
    subprocess.check_call([*cc, *flags, "-Wall", "-shared", "-fPIC", "-I", include, os.path.join(CSRC, "fastcall.c"), "-o", tmp])
    os.replace(tmp, out)
    return out


def tensorcall_built_for(torch) -> str:
    """What _tensorcall.so is good for: it reads tensors through accessors compiled into it, so one build of torch and one Python."""
    return " ".join((torch.__version__, str(torch.version.git_version), sys.implementation.cache_tag))


def build_tensorcall(out: str = TENSORCALL, flags: Sequence[str] = ("-O2",)) -> Optional[str]:
    """The binding's calls from tensors, a CPython extension against torch's own headers.  None where it cannot be built: the
    binding then converts tensors itself."""
    if os.path.exists(out):
        os.remove(out)  # not one of another source
    try:
        import torch
    except ImportError as e:
        print("calls from tensors not built: no torch (%s)" % e)
        return None
    home, include = os.path.dirname(torch.__file__), sysconfig.get_paths()["include"]
    if not all(os.path.exists(f) for f in (os.path.join(include, "Python.h"), os.path.join(home, "include", "c10", "hip", "HIPStream.h"))):
        print("calls from tensors not built: they need the headers of Python and of torch for ROCm")
        return None
    cxx = [shutil.which("g++")] if shutil.which("g++") else [HIPCC]
    tmp, lib = out + ".tmp.%d" % os.getpid(), os.path.join(home, "lib")
    command = [
        *cxx, *flags, "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
        '-DBNN_BUILT_FOR="%s"' % tensorcall_built_for(torch),
        "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I", include, "-I", os.path.join(ROOT, "include"),
        "-isystem", os.path.join(home, "include"), "-isystem", os.path.join(home, "include", "torch", "csrc", "api", "include"),
        "-isystem", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"), os.path.join(CSRC, "tensorcall.cpp"), "-o", tmp,
        "-L", lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath," + lib]
    try:
        subprocess.check_call(command)
    except (OSError, subprocess.CalledProcessError) as e:
        print("calls from tensors not built:", e)
        return None
    os.replace(tmp, out)
    return out


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        tensors = ex.submit(build_tensorcall)
        objs = list(ex.map(_compile, SOURCES))
        tmp = LIB + ".tmp.%d" % os.getpid()
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
        os.replace(tmp, LIB)
        built = [LIB, build_fastcall(), tensors.result()]
    if verbose:
        print("built", *built)
    return LIB


if __name__ == "__main__":
    if "--sanitize" in sys.argv[1:]:
        print("built", build_sanitized())
    else:
        build(verbose=True)

"""Build the HIP library in-tree: paper_2312_08583_amd/libfp6_linear.so (gfx950 only)."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfp6_linear.so")
SOURCES = ["fp6_abi.hip", "fp6_pack.hip", "fp6_decode.hip", "fp6_gemm.hip", "fp6_gemm_variants.hip", "fp6_gemm_bf16.hip",
           "fp6_gemm_heights.hip", "fp6_gemm_heights_v2.hip", "fp6_gemm_heights_fp5_fgq.hip", "fp6_probes.hip"]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
         # packed-fp32 VALU forms are switched off for every kernel of this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def native_path() -> str:
    """Marshalling of the hot-path calls for Python, built for this Python and this torch: no other finds it under this name."""
    import sysconfig
    import torch
    return os.path.join(HERE, "_native-torch" + torch.__version__ + sysconfig.get_config_var("EXT_SUFFIX"))


def build_native() -> str:
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    include, libs = os.path.join(root, "include"), os.path.join(root, "lib")
    path = native_path()
    part = "%s.%d" % (path, os.getpid())          # whole when it appears under its name: other processes may be importing it
    try:
        subprocess.run(["hipcc", "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                        "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
                        "-isystem", include, "-isystem", os.path.join(include, "torch", "csrc", "api", "include"),
                        "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
                        os.path.join(CSRC, "fp6_python.cpp"), "-o", part,
                        "-L" + libs, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], check=True)
        os.replace(part, path)
    finally:
        if os.path.exists(part):
            os.remove(part)
    return path


def build(verbose: bool = False, extra_flags=(), lib: str = LIB, tag: str = "") -> str:
    """Compile every source and link `lib`.  extra_flags / tag are for tuning builds (-D switches)."""
    os.makedirs(OBJ, exist_ok=True)

    def _compile(src: str) -> str:
        obj = os.path.join(OBJ, os.path.splitext(src)[0] + tag + ".o")
        subprocess.run(["hipcc", *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj], check=True)
        return obj

    with ThreadPoolExecutor(max_workers=8) as ex:
        native = ex.submit(build_native) if lib == LIB else None
        objs = list(ex.map(_compile, SOURCES))
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs], check=True)
    if native:
        native.result()
    if verbose:
        print("built", lib)
    return lib


if __name__ == "__main__":
    build(verbose=True)

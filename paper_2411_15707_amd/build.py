"""Compile the HIP sources under csrc/ into paper_2411_15707_amd/libnimbus_cop.so (gfx950), and the module that
calls it from Python without ctypes (csrc/calls.cpp) into paper_2411_15707_amd/_calls<suffix of the interpreter>."""
import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libnimbus_cop.so")
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))     # (of one interpreter)

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_calls() -> str:
    import torch
    from torch.utils import cpp_extension
    flags = ["-std=c++17", "-O2", "-Wall", "-fPIC", "-shared", "-fvisibility=hidden",
             f'-DNIMBUS_TORCH_VERSION="{torch.__version__}"']
    for path in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]:
        flags += ["-isystem", path]
    # (torch's own libraries are in the process already when the module is imported)
    links = ["-L" + path for path in cpp_extension.library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    cxx = os.environ.get("CXX", "g++")
    subprocess.run([cxx] + flags + ["-o", CALLS, os.path.join(CSRC, "calls.cpp")] + links, check=True)
    return CALLS


def build(extra_flags=()) -> str:
    """one object per source, compiled side by side, then one link"""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    srcs = sources()
    with tempfile.TemporaryDirectory(prefix="nimbus_cop_build_") as tmp:
        def compile_one(src):
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            subprocess.run([hipcc] + HIPCC_FLAGS + list(extra_flags) + ["-c", "-o", obj, src], check=True)
            return obj
        with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as pool:
            calls = pool.submit(build_calls)
            objs = list(pool.map(compile_one, srcs))
            calls.result()
        subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, check=True)
    return LIB


if __name__ == "__main__":
    print(build(sys.argv[1:]))

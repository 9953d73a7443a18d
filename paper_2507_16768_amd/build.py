"""Builds libwgrammar.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libwgrammar.so")
SOURCES = ["wg_api.cpp", "wg_lower.cpp", "wg_regex.cpp", "wg_vocab_index.cpp", "wg_kernels.hip", "wg_sample.hip"]
HEADERS = ["wg_internal.h", "wg_buffer.h", "wg_device.h", "wg_launch.h", "wg_order.h", os.path.join("..", "..", "include", "wg.h")]
# a kernel's first dwords of arguments are in scalar registers when its wavefronts begin
PRELOADED_DWORDS = 14
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
         # packed-fp32 instruction selection is switched off for every kernel in this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Xarch_device", "-mllvm=-amdgpu-kernarg-preload-count=%d" % PRELOADED_DWORDS, "-DWG_PRELOADED_DWORDS=%d" % PRELOADED_DWORDS,
         # found by its name next to the Python module, wherever the tree lies
         "-Wl,-soname,libwgrammar.so"]


NATIVE = os.path.join(HERE, "_native.so")      # the Python module behind binding.py, on top of LIB
NATIVE_SOURCE = "wg_python.cpp"


def is_stale():
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in SOURCES + HEADERS + [NATIVE_SOURCE])


def _torch_dir():
    import importlib.util
    return os.path.dirname(importlib.util.find_spec("torch").origin)


def build_native(verbose=False):
    """The Python module: host code only, against torch's headers and LIB."""
    import sysconfig
    torch = _torch_dir()
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = NATIVE + ".%d.tmp" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-isystem", os.path.join(torch, "include"), "-isystem", os.path.join(torch, "include", "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
           "-o", tmp, os.path.join(CSRC, NATIVE_SOURCE), "-L" + HERE, "-l:libwgrammar.so", "-L" + os.path.join(torch, "lib"),
           "-lc10", "-lc10_hip", "-ltorch", "-ltorch_cpu", "-ltorch_python",
           "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + os.path.join(torch, "lib")]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, NATIVE)
    return NATIVE


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".%d.tmp" % os.getpid()
    cmd = [hipcc] + FLAGS + ["-o", tmp] + [os.path.join(CSRC, f) for f in SOURCES]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, LIB)
    build_native(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

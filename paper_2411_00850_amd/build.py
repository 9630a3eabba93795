"""Build libgwq.so (HIP, gfx950 only) with hipcc and the extension module _call.so (C++) in-tree."""
import importlib.metadata
import importlib.util
import os
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libgwq.so")
SOURCES = ["gwq_api.hip", "gwq_pack.hip", "gwq_decode.hip", "gwq_gemm.hip", "gwq_gemm_frag.hip", "gwq_quality.hip", "gwq_score.hip", "gwq_probe.hip"]

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"]


CALL = os.path.join(HERE, "_call.so")                  # Python extension module: the plain gwq.linear call


STAMP_LIB = os.path.join(HERE, "libgwq_stamp.so")     # measurement build: kernels record device timestamps


# Checking build for the CPU side: the host code of the library (argument checks, layout arithmetic, launch planning)
# under clang's address and undefined-behaviour sanitizers, every report fatal; the device code is built as usual.
# GWQ_SANITIZE_HOST=1 makes the binding load it; the Python process needs the sanitizer runtime loaded first:
#   python -m paper_2411_00850_amd.build --sanitize-host
#   LD_PRELOAD="$(/opt/rocm/lib/llvm/bin/clang -print-file-name=libclang_rt.asan-x86_64.so):$LD_PRELOAD" \
#       ASAN_OPTIONS=detect_leaks=0 GWQ_SANITIZE_HOST=1 python -m pytest tests/test_abi.py -q
SAN_LIB = os.path.join(HERE, "libgwq_san.so")
SAN_FLAGS = ["-O1", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=all", "-shared-libsan"]


def build(verbose: bool = False, stamps: bool = False, sanitize_host: bool = False) -> str:
    """Builds libgwq.so; with `stamps` the separate measurement library libgwq_stamp.so instead, whose
    decode kernels record the shader clock at their milestones (gwq_debug_read_stamps); with `sanitize_host`
    the checking build libgwq_san.so."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    out = SAN_LIB if sanitize_host else STAMP_LIB if stamps else LIB
    cmd = [hipcc, *FLAGS, *(SAN_FLAGS if sanitize_host else []), *(["-DGWQ_STAMP"] if stamps else []), "-I", INCLUDE, "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode:
        # the host pass warns that it does not know the packed-fp32 feature; that is harmless
        noise = "is not a recognized feature for this target"
        print("\n".join(l for l in (res.stdout + res.stderr).splitlines() if noise not in l))
    if res.returncode:
        raise RuntimeError("hipcc failed building " + os.path.basename(out))
    if not stamps:
        try:
            build_call(verbose)
        except (ImportError, OSError, RuntimeError) as e:
            warnings.warn(f"_call.so is not built ({e}): the plain gwq.linear call will go through ctypes")
    return out


def built_for() -> str:
    """The Python and the torch whose objects _call.so reads; compiled into it."""
    return f"torch {importlib.metadata.version('torch')}, Python {sys.version_info[0]}.{sys.version_info[1]}"


def build_call(verbose: bool = False) -> str:
    """Builds _call.so against the headers of the installed torch (host code: no GPU compiler).  Where that fails, none is left."""
    if os.path.exists(CALL):
        os.remove(CALL)
    what = built_for()
    torch = os.path.dirname(importlib.util.find_spec("torch").origin)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f'-DGWQ_BUILT_FOR="{what}"',
           "-I", INCLUDE, "-I", os.path.join(torch, "include"),
           "-I", os.path.join(torch, "include", "torch", "csrc", "api", "include"), "-I", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "gwq_call.cpp"), "-L", os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-o", CALL]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode:
        print(res.stdout + res.stderr)
    if res.returncode:
        raise RuntimeError("building " + os.path.basename(CALL) + " failed")
    return CALL


def stale() -> list:
    """Names of the built files that are older than one of their sources or the public header."""
    call = ["gwq_call.cpp"]
    sources = {LIB: [f for f in os.listdir(CSRC) if f not in call], CALL: call}
    return [os.path.basename(built) for built, names in sources.items() if os.path.exists(built) and
            any(os.path.getmtime(d) > os.path.getmtime(built) for d in [os.path.join(CSRC, f) for f in names] + [os.path.join(INCLUDE, "gwq.h")])]


if __name__ == "__main__":
    print(build(verbose=True, stamps="--stamps" in sys.argv, sanitize_host="--sanitize-host" in sys.argv))

"""Compile libtutti (HIP, gfx950) in-tree: paper_2605_03375_amd/libtutti.so.

hipcc cross-compiles without a GPU.  `python -m paper_2605_03375_amd.build` or `build_lib()`.
"""
import importlib.util
import os
import re
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtutti.so")
BENCH_LIB = os.path.join(HERE, "libtutti_bench.so")  # the same sources with the measurement aids compiled in
# Python callables of the per-layer entry points (host code only); the name says which Python it is for
FAST_CALL = os.path.join(HERE, "_fast_call" + sysconfig.get_config_var("EXT_SUFFIX"))
FAST_CALL_DEPS = [os.path.join(CSRC, "fast_call.cpp"), os.path.join(ROOT, "include", "tutti.h")]
SOURCES = [os.path.join(CSRC, "tutti_api.hip"), os.path.join(CSRC, "tutti_host.cpp")]
DEPS = SOURCES + [os.path.join(CSRC, "tutti_kernels.hip.h"), os.path.join(CSRC, "launch_rules.h"),
                  os.path.join(CSRC, "layer_call.h"),
                  os.path.join(ROOT, "include", "tutti.h"),
                  os.path.join(ROOT, "include", "tutti_bench.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
    # no packed-fp32 instructions in any HIP code of this repository
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel's first arguments, up to 14 words, are in scalar registers when a wavefront starts
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
]


def _build(out: str, defines, force: bool, verbose: bool) -> str:
    if not force and os.path.exists(out):
        if os.path.getmtime(out) >= max(os.path.getmtime(p) for p in DEPS):
            return out
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *defines, f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", *SOURCES, "-o", out]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True, cwd=ROOT)
    return out


def _fast_call_is_current(mark: str) -> bool:
    """Newer than its sources, and built for the PyTorch that is installed (fast_call.cpp leaves the mark)."""
    if not os.path.exists(FAST_CALL) or os.path.getmtime(FAST_CALL) < max(os.path.getmtime(p) for p in FAST_CALL_DEPS):
        return False
    with open(FAST_CALL, "rb") as f:
        return b"[torch " + mark.encode() + b"]" in f.read()


def build_fast_call(force: bool = True, verbose: bool = False):
    """The extension module that binding.py calls the per-layer entry points through, or None where PyTorch, Python's headers
    or a C++ compiler are missing: binding.py makes the same calls through ctypes then, and libtutti needs none of them."""
    spec = importlib.util.find_spec("torch")
    include = sysconfig.get_paths()["include"]
    cxx = os.environ.get("CXX", "g++")
    missing = [what for what, there in (("PyTorch", spec is not None), (f"{include}/Python.h",
                                        os.path.exists(os.path.join(include, "Python.h"))),
                                        (cxx, shutil.which(cxx.split()[0]) is not None)) if not there]
    if missing:
        print(f"no extension module for Python calls: {', '.join(missing)} not found", file=sys.stderr)
        return None
    torch = list(spec.submodule_search_locations)[0]
    with open(os.path.join(torch, "version.py")) as f:
        version = re.search(r"__version__ *= *['\"]([^'\"]+)", f.read()).group(1)
    if not force and _fast_call_is_current(version):
        return FAST_CALL
    cmd = [*cxx.split(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
           "-Wno-missing-field-initializers", f'-DBUILT_FOR_TORCH="{version}"', f"-I{os.path.join(ROOT, 'include')}",
           f"-I{include}", "-isystem", os.path.join(torch, "include"),
           "-isystem", os.path.join(torch, "include", "torch", "csrc", "api", "include"), FAST_CALL_DEPS[0],
           "-o", FAST_CALL, f"-L{os.path.join(torch, 'lib')}", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True, cwd=ROOT)
    return FAST_CALL


def build_lib(force: bool = True, verbose: bool = False) -> str:
    """The product library: paper_2605_03375_amd/libtutti.so, and the extension module beside it."""
    lib = _build(LIB, [], force, verbose)
    build_fast_call(force, verbose)
    return lib


def build_bench_lib(force: bool = True, verbose: bool = False) -> str:
    """The measurement library: the same entry points plus baselines, tuning knobs and all launch shapes."""
    return _build(BENCH_LIB, ["-DTUTTI_BENCH_BUILD"], force, verbose)


if __name__ == "__main__":
    print(build_lib(force=True, verbose=True))
    print(build_bench_lib(force=True, verbose=True))

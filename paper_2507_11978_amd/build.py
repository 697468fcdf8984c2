"""Build libnt.so (HIP kernels + C ABI) for gfx950 with hipcc and _nt_calls.so (the binding's native marshalling), in-tree.

Each source is compiled to an object file in parallel (the kernel instantiations are
spread over several translation units for that purpose), then linked."""
from __future__ import annotations

import glob
import importlib.metadata
import importlib.util
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libnt.so")
CALLS = os.path.join(HERE, "_nt_calls.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the epilogues unroll 256 accumulator elements with address arithmetic, masks and format switches per
         # element: above LLVM's default size limit for "#pragma unroll", and a loop left rolled would index
         # the accumulator registers dynamically, i.e. move them to scratch memory
         "-mllvm", "-pragma-unroll-threshold=100000",
         "-Wall", "-Wno-unused-function"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.cpp")) + glob.glob(os.path.join(CSRC, "*.hip")))


def _headers():
    return glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(HERE, "..", "include", "nt.h")]


def _quiet(text: str) -> str:
    # the host pass does not know the device-only target feature and says so; harmless
    return "\n".join(ln for ln in text.splitlines() if "packed-fp32-ops" not in ln)


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    newest = max(os.path.getmtime(p) for p in [src] + _headers())
    if not force and os.path.exists(obj) and os.path.getmtime(obj) >= newest:
        return obj
    res = subprocess.run(["hipcc"] + FLAGS + ["-c", src, "-o", obj], capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n" + _quiet(res.stdout + res.stderr))
    msg = _quiet(res.stdout + res.stderr).strip()
    if msg:
        print(msg, flush=True)
    return obj


def _build_calls(force: bool) -> str | None:
    """The extension module that takes the launching calls' torch tensors apart (host code, for the torch and the Python that are installed).  The
    C library does without it, and so does the binding, through ctypes: where it cannot be built, the reason is returned."""
    src = os.path.join(CSRC, "python", "calls.cpp")
    spec = importlib.util.find_spec("torch")
    if spec is None or not spec.submodule_search_locations:
        return "PyTorch is not installed"
    torch = spec.submodule_search_locations[0]
    try:
        version = importlib.metadata.version("torch")
    except importlib.metadata.PackageNotFoundError:
        version = "unknown"
    built_for, note = f"{version} {sysconfig.get_config_var('EXT_SUFFIX')}", os.path.join(OBJ, "calls.built_for")
    newest = max(os.path.getmtime(p) for p in (src, os.path.join(CSRC, "python", "without_lock.h"), os.path.join(HERE, "..", "include", "nt.h")))
    if not force and os.path.exists(CALLS) and os.path.getmtime(CALLS) >= newest and os.path.exists(note):
        with open(note) as f:
            if f.read() == built_for:
                return None
    include = [os.path.join(torch, "include"), os.path.join(torch, "include", "torch", "csrc", "api", "include"), os.path.join(ROCM, "include"),
               sysconfig.get_paths()["include"]]
    # (the macros select HIP's headers for the AMD compiler and torch's for ROCm, as torch's own extension builder does)
    cmd = (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"] + ["-isystem" + i for i in include] +
           [src, "-o", CALLS, "-L" + os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"])
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        error = res.stdout + res.stderr if res.returncode else None
    except OSError as e:
        error = str(e)
    if error is not None:
        if os.path.exists(CALLS):
            os.remove(CALLS)                               # (built from other sources, or for another torch)
        return f"g++ failed on {src}:\n{error}"
    with open(note, "w") as f:
        f.write(built_for)
    return None


def build(force: bool = True, jobs: int = 8) -> str:
    """Compile every HIP/C++ source into paper_2507_11978_amd/libnt.so, and the binding's extension module beside it if there is a PyTorch to
    build it for.  force=False recompiles only what is older than its source or a header."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        calls = pool.submit(_build_calls, force)
        objs = list(pool.map(lambda s: _compile(s, force), sources()))
        skipped = calls.result()
    res = subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs,
                         capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + _quiet(res.stdout + res.stderr))
    if skipped:
        print(f"{CALLS} not built, calls will be marshalled through ctypes: {skipped}", flush=True)
    return LIB


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv))

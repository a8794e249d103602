"""Build liboasis.so (all HIP kernels + the C ABI) for gfx950 with hipcc, and the binding's native
marshalling (_fastcall.so) with the host compiler, in-tree."""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import warnings

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
LIB_PATH = os.path.join(PKG_DIR, "liboasis.so")


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build liboasis.so)")


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(PKG_DIR, "csrc", "*.hip")))


BUILD_DIR = os.path.join(ROOT, "_build")


def flags() -> list[str]:
    return [
        "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
        # packed-FP32 VALU ops stay disabled in every kernel
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wall", "-Wno-unused-function",
        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG_DIR, "csrc"),
    ]


# Extra compiler flags of single sources. attn.hip: keep MFMA accumulators and
# results in VGPRs; otherwise the compiler parks the attention's accumulators in
# AGPRs and copies all 64 of them to VGPRs on every unit for the rare rescale
# path.
FILE_FLAGS = {"attn.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


FASTCALL_PATH = os.path.join(PKG_DIR, "_fastcall.so")


def rocm_include() -> str:
    """The HIP headers that belong to hipcc."""
    prefixes = [os.environ.get("ROCM_PATH"), *(os.path.dirname(os.path.dirname(p))
                                               for p in (hipcc(), os.path.realpath(hipcc()))), "/opt/rocm"]
    for inc in (os.path.join(p, "include") for p in prefixes if p):
        if os.path.exists(os.path.join(inc, "hip", "hip_runtime_api.h")):
            return inc
    raise RuntimeError("hip/hip_runtime_api.h not found beside hipcc")


def fastcall_cmd(out: str) -> list[str]:
    """The host compiler's command for the extension module (PyTorch's headers and libraries)."""
    import sysconfig
    from torch.utils import cpp_extension as ext
    inc = [*ext.include_paths("cpu"), sysconfig.get_paths()["include"], rocm_include()]
    # NDEBUG also because pybind11's debug reference counter is a thread_local: loading a library that has one
    # leaves every earlier library's thread_local access on glibc's slow path (torch calls about 10 % slower)
    return [os.environ.get("CXX") or "g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-Wall",
            "-DNDEBUG", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I", os.path.join(ROOT, "include"),
            *(f"-isystem{p}" for p in inc), os.path.join(PKG_DIR, "csrc", "fastcall.cpp"), "-o", out,
            *(f"-L{p}" for p in ext.library_paths("cpu")), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def _run(cmd: list[str]) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed ({res.returncode}): {' '.join(cmd)}\n{err}")
    return err


def build_fastcall(out: str) -> tuple[list[str], str, str | None]:
    """Compile the native marshalling: command, compiler output, and what went wrong (None: built)."""
    cmd: list[str] = []
    try:
        cmd = fastcall_cmd(out)
        return cmd, _run(cmd), None
    except (RuntimeError, OSError, ImportError) as e:
        return cmd, "", str(e)


def build(verbose: bool = False) -> str:
    """Compile every HIP source (one hipcc process per file, in parallel) and link liboasis.so next
    to this file; returns its path. The native marshalling beside it needs a host C++ compiler and
    PyTorch's headers; without them the library is built all the same, with a warning, and calls are
    marshalled in Python."""
    from concurrent.futures import ThreadPoolExecutor
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sources()
    objs = [os.path.join(BUILD_DIR, os.path.splitext(os.path.basename(f))[0] + ".o") for f in srcs]
    cmds = [[hipcc(), *flags(), *FILE_FLAGS.get(os.path.basename(f), []), "-c", f, "-o", o]
            for f, o in zip(srcs, objs)]
    try:
        jobs = len(os.sched_getaffinity(0))
    except AttributeError:  # pragma: no cover
        jobs = os.cpu_count() or 1
    fast_tmp = FASTCALL_PATH + ".tmp"
    with ThreadPoolExecutor(max_workers=max(1, min(16, jobs))) as ex:
        fast = ex.submit(build_fastcall, fast_tmp)
        errs = list(ex.map(_run, cmds))
    fast_cmd, fast_err, fast_failed = fast.result()
    cmds.append(fast_cmd)
    errs.append(fast_err)
    tmp = LIB_PATH + ".tmp"
    link = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    errs.append(_run(link))
    if verbose:
        for c in cmds + [link]:
            print(" ".join(c), flush=True)
        err = "\n".join(e for e in errs if e.strip())
        if err:
            print(err, file=sys.stderr)
    # a module left from an earlier build never stands beside the new library
    if os.path.exists(FASTCALL_PATH):
        os.remove(FASTCALL_PATH)
    os.replace(tmp, LIB_PATH)
    if fast_failed is None:
        os.replace(fast_tmp, FASTCALL_PATH)
    else:
        warnings.warn(f"the native marshalling was not built (calls go through the slower Python binding): "
                      f"{fast_failed}", RuntimeWarning, stacklevel=2)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))

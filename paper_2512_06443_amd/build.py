"""Builds libvlut.so (HIP kernels + C ABI) for gfx950 with hipcc and _vlut_torch.so (the binding's calls), in-tree."""
from __future__ import annotations

import os
import shlex
import subprocess
import warnings

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
SRC = os.path.join(_HERE, "csrc", "vlut.hip")
LIB = os.path.join(_HERE, "libvlut.so")
TORCH_SRC = os.path.join(_HERE, "csrc", "torch_calls.cpp")
TORCH_LIB = os.path.join(_HERE, "_vlut_torch.so")
INCLUDE = os.path.join(ROOT, "include")

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
    # packed-FP32 instruction selection is switched off for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off",
]


def build(force: bool = True) -> str:
    """Compiles the library and, where it can, the native form of the binding's calls; returns the library's path.  force=False
    only builds what is missing or stale."""
    csrc = os.path.dirname(SRC)         # vlut.hip includes the kernel headers next to it
    sources = [os.path.join(csrc, f) for f in os.listdir(csrc)] + [os.path.join(INCLUDE, "vlut.h")]
    newest = max(os.path.getmtime(f) for f in sources)

    def stale(path: str) -> bool:
        return force or not os.path.exists(path) or os.path.getmtime(path) < newest

    if stale(LIB):
        hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
        _run([hipcc, *HIPCC_FLAGS, "-I", INCLUDE, SRC, "-o", LIB])
    if stale(TORCH_LIB) or not _built_for_this_torch():
        _build_native()
    return LIB


def _built_for() -> str:
    from .binding import built_for      # (needs torch)
    return built_for()


def _built_for_this_torch() -> bool:
    try:
        with open(TORCH_LIB, "rb") as f:
            return _built_for().encode() in f.read()
    except ImportError:
        return False


def _build_native() -> None:
    """TORCH_LIB, if torch, its headers and a C++ compiler are there.  The calls have a Python form, so that a failure is a warning; a
    file of older sources does not outlive it."""
    try:
        cmd = torch_command()
        if cmd:
            _run(cmd)
        return
    except (ImportError, OSError, RuntimeError) as e:
        why = e
    if os.path.exists(TORCH_LIB):
        os.remove(TORCH_LIB)
    warnings.warn(f"{os.path.basename(TORCH_LIB)} is not built, the binding's calls run in their Python form: {why}", RuntimeWarning, stacklevel=3)


def torch_command():
    """The compiler's command for TORCH_LIB; None with a torch that was not built for ROCm (the calls then run in their Python form)."""
    import sysconfig

    import torch
    if torch.version.hip is None:
        return None
    base = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    inc = [INCLUDE, os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include"),
           os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    # (host code only; torch's libraries are found as the ones that are already loaded)
    return [*shlex.split(os.environ.get("CXX", "g++")), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
            f'-DVLUT_BUILT_FOR="{_built_for()}"', f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *["-I" + d for d in inc], TORCH_SRC, "-o", TORCH_LIB,
            "-L" + os.path.join(base, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def _run(cmd) -> None:
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError(cmd[0] + " failed:\n" + proc.stdout)


if __name__ == "__main__":
    print(build())

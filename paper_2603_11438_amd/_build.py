"""Compile libar.so (HIP for gfx950) in-tree with hipcc, and the native part of
the Python binding with g++."""
from __future__ import annotations

import os
import shutil
import subprocess
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIBDIR = os.path.join(PKG, "_lib")
LIB = os.path.join(LIBDIR, "libar.so")

SOURCES = ["ar_kernels.hip", "ring_lds.hip", "direct.hip", "ar_runtime.cpp", "ar_tuner.cpp", "ar_profile.cpp", "ar_noalloc.hip"]

# -packed-fp32-ops: no packed fp32 instructions in device code.
# -ffp-contract=off / no fast-math: every fp32 add is one IEEE RNE operation.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off", "-fno-fast-math", "-Wall", "-Wno-unused-variable",
    "-Wno-unused-but-set-variable",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libar)")


def build(verbose: bool = False) -> str:
    """Compile every HIP/C++ source of libar into _lib/libar.so, and the native
    part of the Python binding (always rebuilds)."""
    os.makedirs(LIBDIR, exist_ok=True)
    args_job = start_tensor_args()
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as objdir:
        # One compiler per source, at the same time; then one link.
        jobs = []
        for s in SOURCES:
            obj = os.path.join(objdir, s + ".o")
            cmd = [hipcc(), *HIPCC_FLAGS, "-c", "-I", INCLUDE, "-I", CSRC, os.path.join(CSRC, s), "-o", obj]
            jobs.append((obj, subprocess.Popen(cmd, cwd=PKG, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                               text=True)))
        done = [(obj, job.communicate()[0], job.returncode) for obj, job in jobs]
        if not any(rc for _, _, rc in done):
            r = subprocess.run([hipcc(), "--offload-arch=gfx950", "-shared", *[obj for obj, _, _ in done], "-o", tmp],
                               cwd=PKG, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            done.append((tmp, r.stdout, r.returncode))
    # hipcc's host pass does not know the packed-fp32 target feature; that
    # warning is expected and harmless.
    lines = [l for _, out, _ in done for l in (out or "").splitlines() if "packed-fp32-ops" not in l]
    if any(rc for _, _, rc in done):
        raise RuntimeError("libar build failed:\n" + "\n".join(lines))
    if verbose and lines:
        print("\n".join(lines))
    os.replace(tmp, LIB)
    finish_tensor_args(args_job)
    return LIB


TENSOR_ARGS_SRC = os.path.join(CSRC, "tensor_args.cpp")
TENSOR_ARGS = os.path.join(LIBDIR, "_tensor_args.so")


def start_tensor_args() -> subprocess.Popen:
    """Start compiling the native part of the Python binding against torch's
    headers (its symbols come from the torch that the caller has imported)."""
    import sysconfig

    from torch.utils import cpp_extension
    import torch

    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DAR_TORCH_VERSION="{torch.__version__}"',
           "-I", sysconfig.get_paths()["include"],
           *[a for d in cpp_extension.include_paths() for a in ("-I", d)], TENSOR_ARGS_SRC,
           *[a for d in cpp_extension.library_paths() for a in ("-L", d)], "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-o", TENSOR_ARGS + ".tmp"]
    os.makedirs(LIBDIR, exist_ok=True)
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def finish_tensor_args(job: subprocess.Popen) -> str:
    out = job.communicate()[0]
    if job.returncode != 0:
        raise RuntimeError("tensor_args build failed:\n" + (out or ""))
    os.replace(TENSOR_ARGS + ".tmp", TENSOR_ARGS)
    return TENSOR_ARGS


ABI_CHECK_SRC = os.path.join(ROOT, "tests", "native", "abi_gpu_check.cpp")
ABI_CHECK = os.path.join(ROOT, "tests", "native", "abi_gpu_check")


def build_abi_check() -> str:
    """Compile the host program that drives libar through its C ABI alone
    (a GPU test runs it); it links the in-tree libar.so by a relative rpath."""
    rpath = "$ORIGIN/" + os.path.relpath(LIBDIR, os.path.dirname(ABI_CHECK))
    tmp = ABI_CHECK + ".tmp"
    cmd = [hipcc(), "-O2", "-std=c++17", "-Wall", "-I", INCLUDE, ABI_CHECK_SRC, "-L", LIBDIR, "-lar",
           f"-Wl,-rpath,{rpath}", "-o", tmp]
    r = subprocess.run(cmd, cwd=ROOT, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("abi_gpu_check build failed:\n" + (r.stdout or "") + (r.stderr or ""))
    os.replace(tmp, ABI_CHECK)
    return ABI_CHECK


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_abi_check())

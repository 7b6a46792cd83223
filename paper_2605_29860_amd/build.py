"""Builds the HIP shared library for gfx950 with hipcc (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libespo.so")
# translation units: source and its own flags (the step kernels take most of the time, so each logit type is one)
SOURCES = [("espo_step.hip", []), ("espo_step.hip", ["-DESPO_STEP_F32"]), ("espo_advantages.hip", []), ("espo_whiten.hip", []),
           ("espo_batch_stats.hip", []), ("espo_api.hip", [])]
# packed-fp32 VALU forms are switched off for every device translation unit
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               # device code never produces or consumes NaN; this drops the re-quieting of every fmax operand
               "-Xarch_device", "-fno-honor-nans", "-Xarch_device", "-Wno-nan-infinity-disabled"]


def build_library(verbose: bool = False) -> str:
    """Builds libespo.so and, beside it, the module that checks the binding's tensor arguments."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        def run(cmd):
            return subprocess.run(cmd, cwd=tmp, capture_output=True, text=True)

        objs = [os.path.join(tmp, f"{i}.o") for i in range(len(SOURCES))]
        cmds = [[hipcc, *HIPCC_FLAGS, *flags, "-c", os.path.join(CSRC, src), "-o", obj] for (src, flags), obj in zip(SOURCES, objs)]
        with ThreadPoolExecutor(len(cmds) + 1) as pool:
            checker = pool.submit(build_tensor_checker, verbose)
            results = list(pool.map(run, cmds))
            checker.result()
        out = os.path.join(tmp, "libespo.so")
        if all(r.returncode == 0 for r in results):
            results.append(run([hipcc, "--offload-arch=gfx950", "-shared", "-o", out, *objs]))
        for res in results:
            if verbose or res.returncode != 0:
                # the host pass does not know the device-only feature flag; that notice is noise
                print("\n".join(l for l in (res.stdout + res.stderr).splitlines() if "packed-fp32-ops" not in l))
        if any(r.returncode != 0 for r in results):
            raise RuntimeError("hipcc failed building libespo.so")
        os.replace(out, LIB)
    return LIB


TENSOR_SRC = os.path.join(CSRC, "espo_tensor.cpp")
TENSOR_LIB = os.path.join(_HERE, "_espo_tensor.so")


def build_tensor_checker(verbose: bool = False) -> str:
    """Builds the Python module that checks the binding's tensor arguments (host code against torch's headers)."""
    import torch
    home = os.path.dirname(torch.__file__)
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "_espo_tensor.so")
        cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
               f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", "-I" + os.path.join(home, "include"),
               "-I" + os.path.join(home, "include", "torch", "csrc", "api", "include"), "-I" + sysconfig.get_path("include"),
               TENSOR_SRC, "-o", out, "-L" + os.path.join(home, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if verbose or res.returncode != 0:
            print(res.stdout + res.stderr)
        if res.returncode != 0:
            raise RuntimeError("g++ failed building _espo_tensor.so")
        os.replace(out, TENSOR_LIB)
    return TENSOR_LIB


ABI_CHECK_SRC = os.path.join(os.path.dirname(_HERE), "tests", "native", "abi_check.cpp")
ABI_CHECK = os.path.join(os.path.dirname(_HERE), "tests", "native", "abi_check")


def build_abi_check() -> str:
    """Builds the plain HIP host program that drives the C ABI without Python (used by a GPU test)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "-O2", "-std=c++17", ABI_CHECK_SRC, "-o", ABI_CHECK, "-L" + _HERE, "-lespo",
           "-Wl,-rpath,$ORIGIN/../../paper_2605_29860_amd"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        print(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building abi_check")
    return ABI_CHECK


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_abi_check())

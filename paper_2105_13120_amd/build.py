"""Builds the HIP library (csrc/*.hip -> librsa_hip.so) for gfx950 with hipcc, and the Python binding of its main calls
(csrc/binding.cpp -> _binding.so) with the host compiler."""
import glob
import os
import subprocess
import sys
import sysconfig

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
LIB_PATH = os.path.join(_PKG, "librsa_hip.so")
BINDING_PATH = os.path.join(_PKG, "_binding.so")


def sources():
    return sorted(glob.glob(os.path.join(_PKG, "csrc", "*.hip")))


def build_library(verbose=False):
    """Compile every HIP source for gfx950 into one shared library (always recompiles); needs hipcc alone."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [
        hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
        "-I" + os.path.join(_ROOT, "include"), "-I" + os.path.join(_PKG, "csrc"),
        # packed fp32 VALU forms are switched off on the test machines
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wno-unused-command-line-argument",
    ] + sources() + ["-o", LIB_PATH]
    _run(cmd, verbose)
    return LIB_PATH


def build_binding(verbose=False):
    """Compile the binding against the library; needs torch's headers and a host compiler."""
    import torch
    base = os.path.dirname(torch.__file__)
    inc = [os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"],
           os.path.join(_ROOT, "include")]
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
          "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
         + ["-I" + p for p in inc] + [os.path.join(_PKG, "csrc", "binding.cpp"), "-o", BINDING_PATH,
          "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip",
          "-L" + _PKG, "-l:librsa_hip.so", "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + os.path.join(base, "lib")], verbose)
    return BINDING_PATH


def build(verbose=False):
    """Both; the library is there as soon as it is compiled, also where the binding cannot be built."""
    build_library(verbose)
    build_binding(verbose)
    return LIB_PATH


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + res.stdout + res.stderr)


if __name__ == "__main__":
    print(build_library(verbose=True) if sys.argv[1:] == ["--library"] else build(verbose=True))

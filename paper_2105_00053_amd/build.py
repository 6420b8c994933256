"""Builds the HIP library (gfx950) and the host-only check library, in-tree.

    python -m paper_2105_00053_amd.build

Each .hip translation unit is compiled to an object in parallel, then linked
into libpositnn_hip.so next to this file.  Packed-FP32 instruction selection is
switched off for all device code.
"""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpositnn_hip.so")
HOSTCHECK = os.path.join(HERE, "libpositnn_hostcheck.so")
RATES = os.path.join(HERE, "libpositnn_rates.so")  # instruction-issue microbenchmarks for bench.py --issue-rates
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

NATIVE = os.path.join(HERE, "positnn_native.so")  # the binding's marshalling in C++ (csrc/binding_native.cpp)

UNITS = ["api_elementwise.hip", "api_gemm.hip", "direct_gemm.hip", "direct_conv.hip", "api_conv.hip", "api_glue.hip", "api_noquire.hip", "api_loss.hip"]
# Floating-point model, stated rather than left to the compiler's default: the fp64 "buckets" that carry exact
# sums rely on every operation being the IEEE one that is written -- (r + C) - C must round r, not fold to r, and a
# multiply-add is fused only where the source says fma().  So: no fast-math, no contraction across operations.
FP_FLAGS = ["-fno-fast-math", "-ffp-contract=off"]
DEVICE_FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH,
                "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"] + FP_FLAGS + [
                "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        sys.stderr.write(" ".join(cmd) + "\n" + r.stdout + "\n")
        raise RuntimeError("build step failed: " + cmd[-1])
    return r.stdout


def _compile(unit):
    src = os.path.join(CSRC, unit)
    obj = os.path.join(OBJ, unit.replace(".hip", ".o"))
    _run([HIPCC] + DEVICE_FLAGS + ["-c", src, "-o", obj])
    return obj


def _native_command():
    """g++ line of the extension module: against torch's headers and libraries (those that `import torch` has loaded by then).
    None where the compiler or headers are not installed: the binding does without the module."""
    import shutil
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    needed = [os.path.join(sysconfig.get_paths()["include"], "Python.h"), os.path.join(root, "include", "ATen", "ATen.h")]
    if shutil.which("g++") is None or not all(os.path.exists(p) for p in needed):
        return None
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
            "-I" + os.path.join(root, "include"), "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "binding_native.cpp"),
            "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", NATIVE]


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(UNITS) + 1)) as ex:
        command = _native_command()
        native = ex.submit(_run, command) if command else None
        objs = list(ex.map(_compile, UNITS))
        if native:
            native.result()
        else:
            sys.stderr.write("no g++, or no headers of Python or torch: positnn_native.so is left out\n")
            if os.path.exists(NATIVE):
                os.remove(NATIVE)  # built from other sources
    _run([HIPCC, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", LIB] + objs)
    # host-only build of the scalar functions, for CPU unit tests
    _run([HIPCC, "-O2", "-std=c++17", "-fPIC", "-shared", "--cuda-host-only", "-x", "hip"] + FP_FLAGS + [
          "-Wno-unused-command-line-argument", os.path.join(CSRC, "host_check.hip"), "-o", HOSTCHECK])
    _run([HIPCC] + DEVICE_FLAGS + ["-shared", os.path.join(CSRC, "issue_rates.hip"), "-o", RATES])
    if verbose:
        print("built", ", ".join(p for p in (LIB, HOSTCHECK, NATIVE, RATES) if os.path.exists(p)))
    return LIB


if __name__ == "__main__":
    build(verbose=True)

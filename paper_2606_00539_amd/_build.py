"""Builds libgnmr.so (hipcc for gfx950) and the module _calls (gcc) in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libgnmr.so")
SOURCES = [os.path.join(PKG, "csrc", f)
           for f in ("gnmr_runtime.hip", "k1_sumsq.hip", "k23_control.hip", "k123_step.hip",
                     "k4_actuator.hip", "k5_wgrad.hip")]
HEADERS = [os.path.join(PKG, "csrc", f)
           for f in ("gnmr_internal.h", "k1_geometry.h", "k1_item.h", "k3_pool.h", "lane_ops.h",
                     "launch_tag.h", "unit_step.h")] + [os.path.join(ROOT, "include", "gnmr.h")]

# Marshalling of the per-step calls (host code), for the Python that builds it: the
# name carries that Python's ABI, so that no other one loads it.
CALLS = os.path.join(PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
CALLS_SOURCE = os.path.join(PKG, "csrc", "py_calls.c")

# Packed-fp32 instructions are switched off for all device code.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build(verbose: bool = True) -> str:
    cmd = [hipcc(), *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"),
           "-o", LIB + ".tmp", *SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    build_calls(verbose)
    return LIB


def calls_command(out_path: str, *flags: str) -> list:
    return ["gcc", "-O2", "-fPIC", "-shared", "-Wall", *flags, "-I", os.path.join(ROOT, "include"),
            "-I", sysconfig.get_paths()["include"], "-o", out_path, CALLS_SOURCE]


def build_calls(verbose: bool = True) -> str:
    cmd = calls_command(CALLS + ".tmp")
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(CALLS + ".tmp", CALLS)
    untagged = os.path.join(PKG, "_calls.so")   # any Python would load one left by an older build
    if os.path.exists(untagged):
        os.remove(untagged)
    return CALLS


# AddressSanitizer and UndefinedBehaviorSanitizer on the host code only (the
# device code is built as usual); any undefined behaviour aborts.
HOST_SANITIZE_FLAGS = ["-O1", "-g", "-shared-libsan",
                       "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                       "-Xarch_host", "-fno-sanitize-recover=undefined",
                       "-Xarch_host", "-fno-omit-frame-pointer"]


def sanitizer_runtime():
    """The clang AddressSanitizer runtime that a process loading the
    host-sanitized library must preload, or None if this toolchain has none."""
    import glob

    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    found = sorted(glob.glob(os.path.join(rocm, "llvm", "lib", "clang", "*", "lib", "linux",
                                          "libclang_rt.asan-x86_64.so")))
    return found[-1] if found else None


def build_host_sanitized(out_path: str) -> str:
    """libgnmr.so with the host code under the sanitizers, at out_path (for
    CPU tests of the host logic: argument checks, work lists, overlap checks,
    error paths)."""
    cmd = [hipcc(), *HIPCC_FLAGS, *HOST_SANITIZE_FLAGS, "-I", os.path.join(ROOT, "include"),
           "-o", out_path, *SOURCES]
    subprocess.run(cmd, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.PIPE)
    return out_path


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)

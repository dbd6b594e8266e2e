"""Builds libsp.so (the HIP library behind the C ABI of include/sp.h) for gfx950.

Each HIP source is compiled with hipcc for --offload-arch=gfx950 into _build/, then
linked into paper_1110_4623_amd/libsp.so.  Always recompiles.
"""

from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libsp.so")
DEVICE_TESTS = os.path.join(ROOT, "tests", "device")
DEVICE_TESTS_LIB = os.path.join(DEVICE_TESTS, "libsp_device_tests.so")

ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall",
    # code object v5: loadable by the HIP runtime that PyTorch bundles (the process
    # shares that runtime with torch, see _native.py)
    "-mcode-object-version=5",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]
SOURCES = ["sp_api.hip", "sp_barrier.hip", "sp_mutex.hip", "sp_sem.hip", "sp_bench.hip",
           "sp_serve.hip", "sp_cond.hip", "sp_litmus.hip"]


def sources():
    return [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]


def build(verbose: bool = False, save_temps: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    procs = []
    objs = []
    for src in sources():
        obj = os.path.join(BUILD, src.replace(".hip", ".o"))
        cmd = [HIPCC, *CFLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if save_temps:
            cmd.insert(1, "--save-temps")
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, cwd=BUILD, stdout=subprocess.PIPE,
                                            stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l]
        if p.returncode != 0:
            failed.append(src)
            print("\n".join(lines), file=sys.stderr)
        elif verbose and lines:
            print("\n".join(lines))
    if failed:
        raise RuntimeError(f"hipcc failed for {failed}")
    tmp = LIB + ".tmp"
    subprocess.run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp],
                   check=True)
    os.replace(tmp, LIB)
    return LIB


def build_device_tests() -> str:
    """The kernels of tests/device, which use the device headers as a caller's program does."""
    srcs = sorted(os.path.join(DEVICE_TESTS, f) for f in os.listdir(DEVICE_TESTS)
                  if f.endswith(".hip"))
    tmp = DEVICE_TESTS_LIB + ".tmp"
    p = subprocess.run([HIPCC, *CFLAGS, "-shared", *srcs, "-o", tmp], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True)
    if p.returncode != 0:
        print(p.stdout, file=sys.stderr)
        raise RuntimeError("hipcc failed for the device tests")
    os.replace(tmp, DEVICE_TESTS_LIB)
    return DEVICE_TESTS_LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv, save_temps="--save-temps" in sys.argv))

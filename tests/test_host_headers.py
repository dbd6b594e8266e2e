"""The device headers compiled for the CPU, on a host stand-in for their atomics
(tests/host/atomics.hpp): what their waits do when the watchdog has ended the run."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


def build(tmp, source):
    """The headers beside the stand-in that they include in place of their own atomics."""
    sp = tmp / "sp"
    sp.mkdir()
    for name in ("mutex.hpp", "cond.hpp", "semaphore.hpp"):
        shutil.copy(os.path.join(ROOT, "include", "sp", name), sp)
    shutil.copy(os.path.join(HOST, "atomics.hpp"), sp)
    exe = tmp / "prog"
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-g", "-pthread", "-I", str(tmp), "-I",
                           os.path.join(ROOT, "include"), os.path.join(HOST, source), "-o",
                           str(exe)])
    return exe


@pytest.fixture(scope="module")
def unlock_watchdog(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    return build(tmp_path_factory.mktemp("host"), "unlock_watchdog.cpp")


@pytest.mark.parametrize("how", ["unlock", "cond"])
def test_cu_cohort_unlock_ends_with_the_watchdog(unlock_watchdog, how):
    """The holder before on the CU never counts itself complete: the unlock that waits for
    its count ends, with a control block or without, and cond_wait reports the end."""
    p = subprocess.run([str(unlock_watchdog), how], capture_output=True, text=True, timeout=20)
    assert (p.returncode, p.stdout) == (0, "ended\n"), (p.returncode, p.stdout, p.stderr)


def test_reset_list_refuses_one_range_too_many(tmp_path):
    from paper_1110_4623_amd import _native as N
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path / "resets"
    subprocess.check_call([hipcc, "--cuda-host-only", "-x", "hip", "-std=c++17", "-O1", "-w",
                           "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_1110_4623_amd", "csrc"),
                           os.path.join(HOST, "resets.cpp"), "-x", "none", N.LIB_PATH,
                           "-Wl,-rpath," + os.path.dirname(N.LIB_PATH), "-o", str(exe)])
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert (p.returncode, p.stdout) == (0, "refused\n"), (p.returncode, p.stdout, p.stderr)

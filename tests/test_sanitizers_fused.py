"""LDS and buffer accesses of the kernels that run several merge levels at once,
checked on the CPU: ``tests/sanitize/fused_lds_driver.cpp`` includes the device
header as host C++ and runs blocks of every kernel and interval type with the LDS
array and every buffer at its exact size.

Bounds: under AddressSanitizer, every tile of small grids.  The parametrised types
and levels are those a launch can choose, each with all levels stored and with the
last alone, on grids with one window and with several.

Races: under ThreadSanitizer, one block of each with its threads as threads and its
barriers as barriers.  Also a read whose value nothing uses, or a second store of
the same value, counts.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = os.path.join(ROOT, "tests", "sanitize", "fused_lds_driver.cpp")
CLANGXX = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not os.path.exists(CLANGXX), reason="needs the ROCm clang++")


def _run(tmp_path, sanitizer, define):
    exe = tmp_path / "fused_lds"
    # (-O0: a read whose value nothing uses is still made)
    subprocess.run([CLANGXX, "-std=c++17", "-O0", "-g", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-fsanitize=" + sanitizer, define, "-pthread", DRIVER,
                    "-o", str(exe)], check=True, capture_output=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    text = res.stdout[-1500:] + res.stderr[:4000]
    assert "Sanitizer" not in res.stderr and res.returncode == 0, text
    assert "blocks run" in res.stdout, text


def test_every_access_in_bounds(tmp_path):
    _run(tmp_path, "address", "-DBOUNDS")


def test_no_unsynchronised_access(tmp_path):
    _run(tmp_path, "thread", "-DRACES")

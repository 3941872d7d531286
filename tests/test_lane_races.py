"""Shared-memory races between the waves of the register-resident passes, on the host.

tests/native/lane_races.cpp compiles the pass kernels as plain C++ (with the
stand-in header of tests/native/lane_host), runs every kind that has workgroups
of more than one wave lane after lane over three samples, and checks the
recorded shared-memory accesses: no word read by one wave and written by
another between the same two barriers, and the same barriers for every lane.
The memory-access hooks are those of the compiler's thread instrumentation,
linked without its runtime.
"""

import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
NATIVE = os.path.join(HERE, "native")
SIZES = (64, 100, 128, 200, 256, 350, 400, 500, 512, 1000, 1024)


def _clang():
    for c in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib", "llvm", "bin", "clang++"),
              shutil.which("clang++")):
        if c and os.path.exists(c):
            return c
    return None


def test_no_word_is_read_and_written_between_two_barriers(tmp_path):
    cc = _clang()
    if cc is None:
        pytest.skip("clang++ not available")

    def one(n):
        obj, exe = str(tmp_path / f"races{n}.o"), str(tmp_path / f"races{n}")
        r = subprocess.run([cc, "-O1", "-std=c++17", "-w", "-fsanitize=thread", "-I", os.path.join(NATIVE, "lane_host"),
                            f"-DLR_FFT_N={n}", "-c", os.path.join(NATIVE, "lane_races.cpp"), "-o", obj],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
        r = subprocess.run([cc, obj, "-o", exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
        return subprocess.run([exe], capture_output=True, text=True, timeout=300)

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 4)) as ex:
        runs = list(ex.map(one, SIZES))
    for r in runs:
        assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout[-4000:]

"""Rounding of the angular-spectrum transforms against the length's general plan, on the host.

tests/native/as_precision.cpp compiles the device functions of the passes as
plain C++ (stand-in header of tests/native/lane_host), with FMA contraction as
on the device, and compares the r.m.s. error of 1-D transforms with that of the
general plan on the same inputs.
"""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
NATIVE = os.path.join(HERE, "native")
SIZES = (64, 100, 128, 200, 256, 350, 400, 500, 512, 1000, 1024)


@pytest.mark.parametrize("n", SIZES)
def test_no_less_precise_than_the_general_plan(tmp_path, n):
    cc = next((c for c in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib", "llvm", "bin", "clang++"),
                           shutil.which("clang++")) if c and os.path.exists(c)), None)
    if cc is None:
        pytest.skip("clang++ not available")
    exe = str(tmp_path / "as_precision")
    r = subprocess.run([cc, "-O2", "-w", "-mfma", "-ffp-contract=fast", "-std=c++17", "-I",
                        os.path.join(NATIVE, "lane_host"), f"-DLR_FFT_N={n}",
                        os.path.join(NATIVE, "as_precision.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(out.stdout)
    assert out.returncode == 0 and "ALL OK" in out.stdout, out.stdout

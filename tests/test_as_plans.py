"""Host build of the angular-spectrum plans and half-aperture codelets, against direct DFTs."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_as_plans_against_direct_dft(tmp_path):
    cc = next((c for c in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc")
               if c and os.path.exists(c)), None)
    if cc is None:
        pytest.skip("hipcc not available")
    exe = tmp_path / "as_plans_host"
    r = subprocess.run([cc, "-O2", "-std=c++17", os.path.join(HERE, "native", "as_plans_host.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout[-4000:]
    assert "ALL OK" in out.stdout

"""Host logic of the wavelet transform (dwt.hip), compiled into a host program.
Runs on the CPU; needs hipcc to compile the source that holds the kernels."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_forward_scratch_fits_every_plan(tmp_path):
    hipcc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))
                  if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "dwt_host_check")
    res = subprocess.run([hipcc, "-x", "hip", "-O1", "-std=c++17", "--offload-arch=gfx950",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-I", os.path.join(ROOT, "include"),
                          os.path.join(ROOT, "tests", "native", "dwt_host_check.cpp"), "-o", exe],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "all checks passed" in run.stdout, (run.returncode, run.stdout + run.stderr)

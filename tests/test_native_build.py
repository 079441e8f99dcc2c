"""Host logic of the Theta build, compiled from the library's own sources.
Runs on the CPU; needs hipcc to compile against the HIP headers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, name):
    hipcc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))
                  if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / name)
    res = subprocess.run([hipcc, "-x", "hip", "-O1", "-std=c++17", "--offload-arch=gfx950",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-I", os.path.join(ROOT, "include"),
                          os.path.join(ROOT, "tests", "native", name + ".cpp"), "-o", exe],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "all checks passed" in run.stdout, (run.returncode, run.stdout + run.stderr)


def test_only_missing_memory_leaves_the_table_out(tmp_path):
    _run(tmp_path, "try_alloc_check")


def test_weights_table_takes_at_most_an_eighth_of_the_free_memory(tmp_path):
    _run(tmp_path, "table_room_check")

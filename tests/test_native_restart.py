"""The basis change of the Lanczos restart (host code, tridiag.hpp): the kept
vectors are orthonormal, span the top Ritz vectors, and turn the projection and
its coupling to the next Lanczos vector into the returned tridiagonal matrix."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_restart_keeps_the_top_ritz_space_tridiagonal(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "restart_check")
    res = subprocess.run([gxx, "-O2", "-std=c++17", os.path.join(ROOT, "tests", "native", "restart_check.cpp"),
                          "-o", exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0
    lines = out.stdout.strip().splitlines()
    assert len(lines) == 18
    eps = np.finfo(float).eps
    for line in lines:
        f = line.split()
        m, l, bm = int(f[0]), int(f[1]), float(f[2])
        v = np.array([float(x) for x in f[3:]])
        a, b, C, ra, rb = np.split(v, np.cumsum([m, m - 1, m * l, l]))
        C = C.reshape(m, l)
        T = np.diag(a) + np.diag(b, 1) + np.diag(b, -1)
        tol = 100 * m * eps * max(np.max(np.abs(T)) * 2, abs(bm))   # a few roundings per rotation
        assert np.max(np.abs(C.T @ C - np.eye(l))) <= 100 * m * eps
        R = np.diag(ra) + np.diag(rb[:-1], 1) + np.diag(rb[:-1], -1)
        assert np.max(np.abs(C.T @ T @ C - R)) <= tol
        assert np.max(np.abs(T @ C - C @ R)) <= tol          # an invariant space of T
        want = np.zeros(l)
        want[-1] = rb[-1]
        assert np.max(np.abs(bm * C[-1] - want)) <= tol
        assert np.max(np.abs(np.linalg.eigvalsh(R) - np.linalg.eigvalsh(T)[-l:])) <= tol

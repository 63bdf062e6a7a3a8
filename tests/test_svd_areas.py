"""The layout of the SVD's work areas (CPU): tests/svd_areas.cpp against the built library."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2604_03960_amd")


def test_work_areas_are_apart_and_aligned(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "svd_areas")
    cmd = ["hipcc", "--offload-arch=gfx950", "-x", "hip", "-O1", "-std=c++17", "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "svd_areas.cpp"), "-o", exe, "-L", PKG, "-ltna", "-Wl,-rpath," + PKG]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr

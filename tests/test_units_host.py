"""Cuts of the transforms' planes on the host, over all grids that a context takes."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_cut_planes_refuse_no_grid_that_whole_ones_take(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "units")
    subprocess.run([cc, "-O2", "-std=c++17", "-I", os.path.join(HERE, "native", "hip_host"), "-I",
                    os.path.join(ROOT, "paper_1807_04638_amd", "csrc"), os.path.join(HERE, "native", "units_host.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr

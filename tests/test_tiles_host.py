"""Indexes of the semi-Lagrangian tiles and windows and of the stencils' 32-lane row
segments on the host, over edges and remainders of every axis (sanitized)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("source", ["sl_tile_host.cpp", "segments_host.cpp"])
def test_every_point_once_and_neighbours_in_place(source, tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "host")
    subprocess.run([cc, "-O2", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                    os.path.join(HERE, "native", "hip_host"), "-I", os.path.join(ROOT, "paper_1807_04638_amd", "csrc"),
                    os.path.join(HERE, "native", source), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr

"""Tile and window indexes of the semi-Lagrangian kernels on the host, over edges and
remainders of every axis (sanitized)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_tiles_cover_and_windows_hold_the_neighbours(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "sl_tile")
    subprocess.run([cc, "-O2", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                    os.path.join(HERE, "native", "hip_host"), "-I", os.path.join(ROOT, "paper_1807_04638_amd", "csrc"),
                    os.path.join(HERE, "native", "sl_tile_host.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr

"""Boxes of the scatter adjoint: every box that the tile cut lets through (its
cells fit) is staged, whatever its rows are padded to."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2102_12739_amd", "csrc")


@pytest.mark.parametrize("box_bytes", [8192, 12288, 16384, 18432])
def test_boxes_whose_cells_fit_fit_with_their_padding(tmp_path, box_bytes):
    exe = tmp_path / "box_pitch_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC,
                    os.path.join(ROOT, "tests", "cpp", "box_pitch_check.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(box_bytes // 32)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    n, padded = map(int, r.stdout.split())
    assert n > padded > n // 4      # some have no room for the padding, many do

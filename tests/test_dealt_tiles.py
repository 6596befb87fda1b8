"""Shares of a tile list that are dealt round-robin, up to the last tile an int
can name (degrid_execute_noalloc takes that many)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2102_12739_amd", "csrc")
TOP = 2 ** 31 - 1


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("dealt") / "next_dealt_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", os.path.join(ROOT, "tests", "cpp", "next_dealt_check.cpp"),
                    "-o", str(out)], check=True)
    return str(out)


@pytest.mark.parametrize("begin,stride,end", [
    (0, 4, 0), (0, 4, 1), (3, 4, 16), (3, 4, 15), (0, 1, 5), (TOP, 512, TOP), (TOP - 1, 512, TOP),
    (TOP - 512, 512, TOP), (TOP - 513, 512, TOP), (TOP - 5000, 512, TOP),
])
def test_a_dealt_share_ends_at_the_last_tile(exe, begin, stride, end):
    r = subprocess.run([exe, str(begin), str(stride), str(end)], capture_output=True, text=True, check=True, timeout=60)
    assert [int(x) for x in r.stdout.split()] == list(range(begin, end, stride))

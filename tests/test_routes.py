"""The host-side launch rules (paper_2403_04206_amd/csrc/grawa_route.h, no GPU dependency) at sizes that no test can
allocate: a small program prints what the rules give."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("route") / "route_driver")
    res = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I",
                          os.path.join(ROOT, "paper_2403_04206_amd", "csrc"), os.path.join(ROOT, "tests", "route_driver.cpp"),
                          "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return lambda *args: [[int(v) for v in line.split()] for line in
                          subprocess.run([out] + [str(a) for a in args], capture_output=True, text=True,
                                         check=True).stdout.splitlines()]


def test_row_split_grid_within_the_launch_limit(driver):
    P = [1, 256, 257, (1 << 26) - 1, 1 << 26, (1 << 26) + 1, (1 << 30) - 256, 1 << 30, (1 << 30) + 1, (1 << 31) + 5, (1 << 32) - 512]
    cells = [(p + 255) // 256 for p in P]
    for n, gx, gy, threads in driver("split", *cells):
        assert gx * threads < 1 << 32 and gy < 1 << 16
        assert n <= gx * gy < n + gy                     # every cell, and less than one block per row for nothing
        assert gy == 1 or n > 1 << 18


def test_no_arrivals_with_many_layers(driver):
    # one arrival per layer on one address: bounded by a rule on the layer count, whatever else the problem is
    assert driver("model", 1, 62, 100, 101, 161, 291, 100000) == [[1, 1], [62, 1], [100, 1], [101, 0], [161, 0], [291, 0], [100000, 0]]

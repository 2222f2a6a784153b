"""Tile of the grad_W_s product (grad_W_tile in csrc/kd_launch.h, compiled for the host), at chunks where the one taken measured at
least 10 % ahead of the next: few tiles, whose rounds of workgroups decide, and many."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2603_01875_amd/csrc/kd_launch.h"
#include <cstdio>
#include <cstdlib>
int main(int, char** a) { std::printf("%%d", kd::grad_W_tile(std::atoll(a[1]), std::atoll(a[2]), kd::kNumCU)); }
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("gw")
    (d / "g.cpp").write_text(PROGRAM % ROOT)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", str(d / "g.cpp"), "-o", str(d / "g")],
                   check=True)
    return str(d / "g")


@pytest.mark.parametrize("H_s, width, rows", [
    (448, 10640, 128),        # 53 us; 75 with 256
    (512, 8192, 128),         # 2.89 ms a call; 4.38 with 256
    (320, 8192, 128), (1344, 1136, 128), (3712, 1888, 128), (448, 16384, 128), (1472, 7248, 192), (3584, 9720, 192),
    (1152, 11224, 256), (2432, 15968, 256)])
def test_the_faster_tile_is_taken(program, H_s, width, rows):
    assert int(subprocess.run([program, str(H_s), str(width)], check=True, capture_output=True, text=True).stdout) == rows

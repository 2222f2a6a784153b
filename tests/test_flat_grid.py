"""Grids of workgroups numbered in a row (flat_grid in csrc/kd_launch.h, compiled for the host): all workgroups are there, and no
axis has 2^32 threads, up to what the widest operand copies and the transposed hidden states of 2^22 tokens take."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2603_01875_amd/csrc/kd_launch.h"
int main() {
  const int64_t T = 1 << 22, edge = 1 << 21;
  const int64_t groups[] = {1, 2, 255, edge - 1, edge, edge + 1, 3 * edge, 3 * edge + 5,
                            T / 64 * (8192 / 32) / 4 + 1,                   /* packed copies of 8192 elements a token */
                            T / 64 * (196608 / 32) / 4, 1 + T / 64 * (65536 / 64)};
  for (int64_t n : groups) {
    const kd::FlatGrid g = kd::flat_grid(n);
    const int64_t all = (int64_t)g.x * g.y;
    if (all < n || all - n >= g.x || (int64_t)g.x * 1024 >= (int64_t)1 << 32 || g.y > 65535 || (n <= edge && g.y != 1)) return 1;
  }
  return 0;
}
"""


def test_flat_grids_hold_all_workgroups(tmp_path):
    src, exe = tmp_path / "g.cpp", tmp_path / "g"
    src.write_text(PROGRAM % ROOT)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0

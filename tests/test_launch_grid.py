"""Grids of the flat selection's scans, compiled for the CPU: inside the launch
limits over all rows and heads that the ABI takes, and every tile once."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_31093_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "launch_grid.h"
int main() {
  const long long max_rows = (1LL << 23) - 1;
  for (long long nq : {1LL, 31LL, 32LL, 33LL, 4097LL, 32768LL * 32, 32768LL * 32 + 1, 32768LL * 64 + 31, max_rows})
    for (int bh : {1, 2, 8, 512, 65535})
      for (int tile : {32, 128, 256}) {
        const long long tiles = (nq + tile - 1) / tile;
        const pisa::HeadGrid g = pisa::head_grid(tiles, bh);
        if (g.x != static_cast<unsigned>(bh) || 256ULL * g.x >= 1ULL << 32 || !g.y || g.y > 65535 || !g.z || g.z > 65535)
          return printf("limits: %lld rows, %d heads\n", nq, bh), 1;
        if (1LL * g.y * g.z < tiles || 1LL * g.y * (g.z - 1) >= tiles) return printf("cover: %lld rows\n", nq), 1;
      }
  return 0;
}
"""


def test_head_grid(tmp_path):
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout

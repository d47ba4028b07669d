"""The waves of a wide sparse x dense product take every (unit, chunk) pair
once and stop, up to the most pairs that the kernel is launched for (CPU: the
kernel's own walk, compiled for the host)."""

import os
import subprocess

import pytest

from paper_1512_00066_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "spmm_plan.hpp"

// Pairs taken by the listed waves; each of them at most once.
static int64_t pairs(uint32_t nunits, uint32_t nch, uint32_t grid, uint32_t from, uint32_t to, bool by_unit, bool mark) {
  std::vector<uint8_t> seen(mark ? (size_t)nunits * nch : 0);
  int64_t n = 0;
  for (uint32_t w = from; w < to; w++) {
    srtc::UnitTurns t(nunits, nch, grid, 4, w / 4, w % 4, by_unit);
    int32_t u, c;
    for (int64_t k = 0; t.next(&u, &c); k++, n++) {
      if (u < 0 || c < 0 || u >= (int64_t)nunits || c >= (int64_t)nch) return printf("out of range: %d %d\n", u, c), -1;
      if (k > (int64_t)nunits * nch) return printf("does not end\n"), -1;
      if (mark && seen[(size_t)c * nunits + u]++) return printf("twice: %d %d\n", u, c), -1;
    }
  }
  return n;
}

int main() {
  const uint32_t shapes[][3] = {{1, 1, 1}, {7, 3, 2}, {100, 7, 8}, {33, 8, 8}, {33, 17, 16}, {5, 9, 24}, {300, 64, 2048}};
  for (bool by_unit : {false, true})
    for (auto &q : shapes) {
      const int64_t n = pairs(q[0], q[1], q[2], 0, q[2] * 4, by_unit, true);
      if (n != (int64_t)q[0] * q[1]) return printf("%u x %u: %lld\n", q[0], q[1], (long long)n), 1;
    }
  // where chunks share lines of X, neighbouring waves take one unit's chunks
  for (uint32_t w = 0; w < 10; w++) {
    srtc::UnitTurns t(100, 5, 40, 4, w / 4, w % 4, true);
    int32_t u = -1, c = -1;
    if (!t.next(&u, &c) || u != (int32_t)(w / 5) || c != (int32_t)(w % 5)) return printf("order: %d %d\n", u, c), 1;
  }
  // the largest products: the turn after a wave's last lies past 2^31
  const uint32_t grid = 2048;
  for (uint32_t nch : {1u, 7u, 8u, 15u})
    for (uint32_t w : {0u, 5000u, grid * 4 - 1}) {
      const uint32_t nunits = 0x7fffffffu / nch;
      const int64_t n = pairs(nunits, nch, grid, w, w + 1, w == 5000, false);
      if (n < 0) return 1;
      if (n < (int64_t)nunits * nch / (grid * 4) - 2) return printf("left out: %u chunks, %lld\n", nch, (long long)n), 1;
    }
  return 0;
}
"""


def test_every_pair_once(tmp_path):
    src, exe = tmp_path / "turns.hip", tmp_path / "turns"
    src.write_text(PROGRAM)
    r = subprocess.run([B.HIPCC, "-O2", "-std=c++17", f"--offload-arch={B.ARCH}", "-x", "hip", "-I", B.CSRC, str(src),
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr

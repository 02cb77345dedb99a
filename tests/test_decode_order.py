"""The decode launch takes every head once for each split, in an order turned with the split
(host code: the header is compiled on its own)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "hk_turn.h"

#include <cstdio>
#include <initializer_list>

int main() {
  long bad = 0, seen = 0;
  for (int n = 1; n <= 17000; n = n < 300 ? n + 1 : n + 167) {
    const uint32_t m = hk::turn_magic(n);
    for (int i = 0; i < 60; ++i) {
      // multiples of n and their neighbours, and the last turns below 2^16
      const long q = i < 40 ? i * 1637L / 40 : 65535 / n - (i - 40);
      for (long h = q * n - 1; h <= q * n + 1; ++h) {
        if (h < 0 || h > 65535) continue;
        for (int x : {0, 1, n / 2, n - 1}) {
          if (x >= n) continue;
          bad += hk::head_of(x, (int)h, n, m) != (x + h) % n;
          ++seen;
        }
      }
    }
  }
  std::printf("%ld %d\n", bad, seen > 100000);
}
"""


def test_every_head_once(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "turn.cpp", tmp_path / "turn"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2606_28831_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    assert out.split() == ["0", "1"]

"""The dynamic-LDS limit of a kernel never falls below what an earlier launch was granted, also
when two host threads raise it at once (host code: the header is compiled on its own)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# One thread is inside its own set(90) when another asks for 152; the first waits (at most a
# second) for the second to be done, so that its own smaller limit is the last one set if the two
# calls can overlap.
PROGRAM = r"""
#include "hk_lds_limit.h"

#include <chrono>
#include <cstdio>
#include <future>
#include <thread>

int main() {
  hk::LdsLimit limit(64);
  size_t now = 64, calls = 0;
  std::promise<void> inside, done;
  auto seen = inside.get_future();
  auto other = done.get_future();
  std::thread small([&] {
    limit.raise(90, [&](size_t b) {
      inside.set_value();
      other.wait_for(std::chrono::seconds(1));
      now = b;
      ++calls;
    });
  });
  seen.wait();
  limit.raise(152, [&](size_t b) { now = b; ++calls; });
  done.set_value();
  small.join();
  const size_t raced = now;
  for (size_t b : {64, 90, 100, 152}) limit.raise(b, [&](size_t x) { now = x; ++calls; });
  const size_t same = calls;
  limit.raise(160, [&](size_t x) { now = x; ++calls; });
  std::printf("%zu %zu %zu %zu\n", raced, same, now, calls);
}
"""


def test_limit_never_falls(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-pthread", "-I" + os.path.join(ROOT, "paper_2606_28831_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    assert out.split() == ["152", "2", "160", "3"]

"""Deferred bookkeeping's records on the host, compiled on their own: every layer of a launch is waited for exactly until it
has been, wherever the launch starts (up to the last of 256 layers) and however many layers it takes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "ckv_books.h"
int main() {
  for (int n_cu : {256, 304, 80, 1}) {
    for (int units = 1; units <= 512; ++units) {
      const int group = ckv::book_group(n_cu, units);
      if (group < 8 || group > 32) return std::printf("group of %d\n", group), 1;
      for (int layers : {1, 8, 40, 256}) {
        ckv::PendingBooks books;
        books.reset(layers);
        for (int first = 0; first < layers; first += group) books.record(first, std::min(group, layers - first));
        // one layer: its own launch, once
        for (int l = layers - 1; l >= 0; l -= 7) {
          int waits = 0, on = -1;
          auto wait = [&](int first) { ++waits; on = first; return 0; };
          books.join(l, wait);
          books.join(l, wait);
          if (waits != 1 || on != l / group * group) return std::printf("%d layers, groups of %d: layer %d waited %d times, on %d\n", layers, group, l, waits, on), 1;
        }
        // the others, then nothing is left
        int waits = 0;
        auto count = [&](int) { ++waits; return 0; };
        books.join(-1, count);
        const int want = layers - (layers + 6) / 7;
        if (waits != want) return std::printf("%d layers, groups of %d: %d waits, %d expected\n", layers, group, waits, want), 1;
        books.join(-1, count);
        if (waits != want) return std::printf("waited again\n"), 1;
      }
    }
  }
  return 0;
}
"""


def test_every_layer_of_a_launch_is_waited_for(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "books.cpp", tmp_path / "books"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2601_16986_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout

"""Choices by size that kernels and host share (ckv_plan.h), compiled on their own."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "ckv_plan.h"\nint main() {\n' + body + "\n  return 0;\n}\n")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2601_16986_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout


def test_logits_are_asked_for_in_portions_that_divide_a_thread_s_groups(tmp_path):
    """The last portion would otherwise go beyond the thread's values."""
    _run(tmp_path, r"""
  for (int groups : {1, 2, 3, 4, 8})
    for (int threads : {256, 512, 1024})
      for (bool lean : {false, true}) {
        const int n = ckv::logit_groups(groups, threads, lean);
        if (n < 1 || groups % n != 0) return std::printf("%d of %d groups, %d threads\n", n, groups, threads), 1;
      }""")


def test_counters_are_looked_at_early_only_if_every_workgroup_runs_at_once(tmp_path):
    _run(tmp_path, r"""
  for (int n_cu : {256, 80})
    for (long long workgroups : {1ll, 10ll, n_cu - 1ll, n_cu + 0ll, n_cu + 1ll, 100000ll})
      if (ckv::looks_early(workgroups, n_cu) != (workgroups < n_cu)) return std::printf("%lld workgroups, %d compute units\n", workgroups, n_cu), 1;""")

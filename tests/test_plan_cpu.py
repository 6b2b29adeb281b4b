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
    for (long long workgroups : {1ll, 10ll, n_cu + 0ll, n_cu + 1ll, 2ll * n_cu, 2ll * n_cu + 1, 100000ll})
      for (bool one_block : {true, false})
        if (ckv::looks_early(workgroups, one_block, n_cu) != (workgroups <= (one_block ? 1 : 2) * n_cu))
          return std::printf("%lld workgroups, %d compute units\n", workgroups, n_cu), 1;""")


def test_attention_only_steps_do_not_wait_for_idle_workgroups(tmp_path):
    """Shapes measured both ways; one launch where the capacity leaves no workgroup idle (unless units are short and many), two where it leaves two or
    more per compute unit."""
    _run(tmp_path, r"""
  struct { int mean, count, cap; bool apart; } measured[] = {
      {1512, 2, 8192, false}, {1112, 32, 1184, false}, {712, 56, 768, false}, {712, 64, 4096, true}, {712, 64, 32768, true}, {1512, 8, 32768, true},
      {1112, 128, 4096, false}, {712, 256, 4096, true}, {1512, 400, 32768, true}, {369, 256, 416, false}, {190, 128, 448, false}, {190, 400, 448, true},
      {690, 64, 1408, false}, {390, 104, 832, false}, {1090, 256, 2240, true}, {2590, 200, 5248, false}, {1590, 32, 3200, false},
      {680, 480, 704, true}, {390, 400, 416, true}, {690, 256, 704, false}, {1590, 400, 1600, false}};
  for (auto& m : measured)
    if (ckv::attends_apart(m.mean, m.count, m.cap, 256) != m.apart) return std::printf("%d units of %d at capacity %d\n", m.count, m.mean, m.cap), 1;
  for (int mean = 1; mean < 32768; mean = mean * 3 / 2 + 1)
    for (int count = 1; count < 2000; count = count * 3 / 2 + 1)
      for (int cap = (mean + 32) / 32 * 32; cap <= 32768; cap = cap * 2 / 32 * 32) {
        const bool one_block = ckv::one_block_each(mean, count, 256);
        const long long idle = (long long)count * (ckv::step_pieces(cap, one_block) - ckv::step_pieces(mean, one_block));
        const bool short_and_many = !one_block && count > 256 && cap <= 2048 && mean <= 768;
        if ((idle == 0 || idle >= 512) && ckv::attends_apart(mean, count, cap, 256) != (idle != 0 || short_and_many)) return std::printf("%d units at %d\n", count, cap), 1;
      }""")


def test_bookkeeping_in_the_step_or_apart(tmp_path):
    """Shapes measured both ways, and the bound that the registers of the one kernel set."""
    _run(tmp_path, r"""
  struct { int mean, count, cap; bool apart; } measured[] = {
      {200, 64, 6144, true}, {200, 256, 6144, true}, {200, 256, 2048, true}, {200, 52, 6144, false}, {200, 256, 256, false}, {700, 128, 6144, false},
      {1200, 104, 6144, false}, {600, 200, 2432, false}, {3700, 64, 3712, true}, {3700, 72, 3712, true}, {5900, 56, 5920, true}, {5900, 32, 5920, false},
      {5900, 104, 5920, false}, {2000, 72, 6144, false}, {2000, 128, 2016, false}, {128, 2, 160, false}, {2048, 8, 8224, true}};
  for (auto& m : measured)
    if (ckv::books_apart(m.mean, m.count, m.cap, 256, 512, 6144) != m.apart) return std::printf("%d units of %d at capacity %d\n", m.count, m.mean, m.cap), 1;
  for (int mean = 1; mean < 32768; mean = mean * 3 / 2 + 1)
    for (int count = 1; count < 2000; count = count * 3 / 2 + 1)
      for (int cap : {6176, 8192, 32768})
        if (!ckv::books_apart(mean, count, cap, 256, 512, 6144)) return std::printf("%d units at %d\n", count, cap), 1;""")


def test_only_large_layers_are_loaded_past_the_caches(tmp_path):
    """Admissions measured both ways, and the last cache's 256 MiB of keys and values as the line."""
    _run(tmp_path, r"""
  struct { long long units, length; bool past; } measured[] = {
      {4, 777, false}, {32, 777, false}, {8, 9350, false}, {32, 3000, false}, {128, 2048, false}, {32, 9350, false}, {48, 9350, false},
      {512, 1024, true}, {64, 9350, true}, {128, 9350, true}, {64, 8191, false}, {64, 8192, true}};
  for (auto& m : measured)
    if (ckv::loads_past_caches(m.units * m.length) != m.past) return std::printf("%lld units of %lld\n", m.units, m.length), 1;""")

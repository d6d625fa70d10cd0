"""The dynamic LDS sizes that follow a call's data (launch_sizes.h), built with
g++: large enough, within the limit, and only a few distinct ones over every
query length and vocabulary, since each takes an entry of the residency table."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <set>
#include <stdio.h>
#include "launch_sizes.h"
int main() {
  std::set<int> words;
  for (int h = 1; h <= 512; ++h) {
    const int w = lcemd::bf16_layout_words(h, 512);
    if (w < h || w > 512) return 1;
    words.insert(w);
  }
  const size_t max = 160 * 1024;
  std::set<size_t> bytes;
  for (size_t b = 1; b <= max; ++b) {
    const size_t r = lcemd::lds_launch_bytes(b, max);
    if (r < b || r > max) return 2;
    bytes.insert(r);
  }
  printf("%zu %zu\n", words.size(), bytes.size());
  return 0;
}
"""


def test_few_distinct_sizes(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "sizes.cpp", str(tmp_path / "sizes")
    src.write_text(PROGRAM)
    cmd = [gxx, "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1812_02091_amd", "csrc"), str(src),
           "-o", exe]
    b = subprocess.run(cmd, capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.returncode
    words, sizes = map(int, r.stdout.split())
    # four bf16 table kernels and two LDS kernels: well within the table
    assert 4 * words + 2 * sizes <= 64, (words, sizes)

"""The step through a leaf's triangle records (rt_layout.h), compiled for the
host: every leaf of 1 to 15 records, also one that ends with the last record
that an accel may hold, is walked record by record and then over."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_00292_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include "rt_layout.h"
int main() {
  int failures = 0;
  for (uint32_t count = 1; count <= RT_MAX_LEAF_SIZE; ++count) {
    const uint32_t last = RT_MAX_TRI_RECORDS - count;
    const uint32_t firsts[] = {0u, 1u, 12345u, last / 2u, last - 1u, last};
    for (uint32_t first : firsts) {
      uint32_t leaf = rt_make_leaf(first, count) & ~RT_LEAF_BIT, k = 0;
      for (; leaf != 0u && k <= count; ++k, leaf = rt_leaf_rest(leaf))
        if (k == count || (leaf & RT_LEAF_FIRST_MASK) != first + k) break;
      if (k != count || leaf != 0u) {
        std::printf("first %u count %u: record %u is %u\n", first, count, k, leaf & RT_LEAF_FIRST_MASK);
        ++failures;
      }
    }
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
"""


def test_leaf_walk(tmp_path):
    src = tmp_path / "leaf.cpp"
    src.write_text(SOURCE)
    exe = str(tmp_path / "leaf")
    b = subprocess.run(["g++", "-std=c++17", "-Wall", f"-I{CSRC}", str(src), "-o", exe],
                       capture_output=True, text=True, timeout=120)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout

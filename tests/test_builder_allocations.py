"""Host allocations of the tree builder (CPU): the collapse of a binary tree to
4-wide nodes holds its pending children in arrays of fixed size, so a node
costs the vectors of its children (three to hold four of them, one of their
numbers) and no list besides."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_00292_amd", "csrc")

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <new>
#include "bvh_build.h"
static long count = 0;
void* operator new(size_t s) {
  ++count;
  if (void* p = std::malloc(s)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
int main() {
  const uint32_t n = 100;
  std::vector<float> V;
  std::vector<uint32_t> I;
  for (uint32_t y = 0; y <= n; ++y)
    for (uint32_t x = 0; x <= n; ++x)
      for (float c : {x / (float)n, y / (float)n, 0.1f * std::sin(0.3f * x) * std::cos(0.2f * y)}) V.push_back(c);
  for (uint32_t y = 0; y < n; ++y)
    for (uint32_t x = 0; x < n; ++x) {
      const uint32_t a = y * (n + 1) + x;
      for (uint32_t i : {a, a + 1, a + n + 1, a + 1, a + n + 2, a + n + 1}) I.push_back(i);
    }
  rtb::BuildInput in{V.data(), I.data(), (uint32_t)V.size() / 3, (uint32_t)I.size() / 3};
  rtb::WideTree t;
  std::string err;
  count = 0;
  if (!rtb::build_mesh(in, 4, 4, t, err, 1)) return 2;
  std::printf("%u nodes, %ld allocations\n", t.node_count, count);
  return count > 4L * t.node_count + 256;
}
"""


def test_collapse_allocations(tmp_path):
    src = tmp_path / "alloc.cpp"
    src.write_text(SOURCE)
    exe = str(tmp_path / "alloc")
    b = subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", str(src), os.path.join(CSRC, "bvh_build.cpp"),
                        "-o", exe, "-lpthread"], capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout

"""The rules that size a traversal launch (rt_launch.h), compiled for the host."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_00292_amd", "csrc")


def run_driver(tmp_path, source):
    src = tmp_path / "driver.cpp"
    src.write_text(source)
    exe = str(tmp_path / "driver")
    b = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", f"-I{CSRC}", f"-I{ROOT}/include", str(src), "-o", exe],
                       capture_output=True, text=True, timeout=120)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout[-3000:]


NOALLOC = r"""
#include <cstdio>
#include <initializer_list>
#include "rt.h"
#include "rt_launch.h"
int main() {
  const size_t limit = RT_NOALLOC_SCRATCH_BYTES / 4, array = rtk_noalloc_array(limit);
  const uint32_t stacks[] = {8, 16, 32}, groups[] = {64, 128, 256}, rays[] = {1, 65, 1000003, 0x7FFFFFFF};
  int failures = 0;
  long taken = 0;
  for (uint32_t s : stacks)
    for (uint32_t wg : groups)
      for (uint32_t n : rays)
        for (uint32_t refill : {1u, 32u, 64u})
          for (uint32_t bound = 1; bound < 300000; ++bound) {
            if (rtk_noalloc_budget(n, refill, s, wg, bound) > limit) break;
            ++taken;
            if (kRtCounterWords + rtk_spill_words(bound, s, false, 0) * wg > array) {
              std::printf("stack %u workgroup %u rays %u bound %u\n", s, wg, n, bound);
              ++failures;
            }
          }
  std::printf("%ld taken, %d failures\n", taken, failures);
  return failures != 0 || taken < 100000;
}
"""


def test_noalloc_scratch_holds_every_launch_taken(tmp_path):
    """A launch within the published limit fits the fixed array with at least
    one workgroup, up to the deepest stack bound that the limit takes."""
    run_driver(tmp_path, NOALLOC)

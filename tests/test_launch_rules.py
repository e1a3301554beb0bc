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
            if (kRtCounterWords + rtk_spill_words(bound, s, false, 0, 4) * wg > array) {
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


RAYS = r"""
#include <cstdio>
#include <initializer_list>
#include <random>
#include <vector>
#include "rt_launch.h"

static int failures = 0;
static void bad(const char* what, uint32_t n, uint32_t wg, uint32_t blocks) {
  if (++failures < 20) std::printf("%s: rays %u workgroup %u blocks %u\n", what, n, wg, blocks);
}

// the same place in 64 bits
static uint64_t place(uint32_t shift, uint64_t v, uint64_t p) {
  return ((((p >> shift) * kRtQueues) + v) << shift) + (p & ((1ull << shift) - 1));
}

// order 0: the waves take chunks in turn; 1: one wave after another takes all
// it may; 2: at random
static void hand_out(uint32_t n, uint32_t wg, uint32_t max_blocks, int order) {
  const LaunchShape s = launch_shape(n, wg, max_blocks);
  const uint32_t wpb = wg / 64u, waves = s.blocks * wpb;
  if (s.blocks < 1 || s.blocks > max_blocks) return bad("blocks", n, wg, max_blocks);
  const uint32_t unit = s.chunk ? s.chunk : s.share;
  std::vector<uint8_t> given((size_t)n / unit + 1, 0);
  std::vector<uint32_t> ranges(waves, 0);
  auto give = [&](uint32_t first) {
    if (first >= n) return;
    if (first % unit || given[first / unit]) return bad("a ray twice", n, wg, max_blocks);
    given[first / unit] = 1;
  };
  for (uint32_t w = 0; w < waves; ++w) {
    give(rt_first_ray(w / wpb, w % wpb, s.blocks, wpb, s.share, s.chunk, s.tile_shift));
    ranges[w] = 1;
  }
  if (s.chunk) {
    if (s.share != s.chunk || (1u << s.tile_shift) % s.chunk) return bad("tile", n, wg, max_blocks);
    uint32_t head[kRtQueues] = {};
    std::mt19937 rng(n ^ wg);
    std::vector<uint32_t> open(waves);
    for (uint32_t w = 0; w < waves; ++w) open[w] = w;
    size_t at = 0;
    while (!open.empty()) {
      if (order == 2) at = rng() % open.size();
      else if (at >= open.size()) at = 0;
      const uint32_t w = open[at];
      bool got = false;
      for (uint32_t k = 0; k < kRtQueues && !got && ranges[w] < kRtRangesPerWave; ++k) {
        const uint32_t v = ((w / wpb) + k) % kRtQueues;
        const uint32_t first = rt_ray_at(s.tile_shift, v, rt_shared_out(s.blocks, wpb, s.share, v) + head[v]);
        if (first >= n) continue;
        head[v] += s.chunk;
        give(first);
        ++ranges[w];
        got = true;
      }
      if (!got) {
        open[at] = open.back();
        open.pop_back();
      } else if (order == 0) {
        ++at;
      }
    }
  }
  for (size_t k = 0; k * unit < n; ++k)
    if (!given[k]) return bad("a ray left out", n, wg, max_blocks);
}

// no position that a head can reach wraps around 2^32
static void heads(uint32_t n, uint32_t wg, uint32_t max_blocks) {
  const LaunchShape s = launch_shape(n, wg, max_blocks);
  if (!s.chunk) return;
  const uint32_t wpb = wg / 64u, waves = s.blocks * wpb;
  for (uint32_t v = 0; v < kRtQueues; ++v) {
    const uint64_t tile = 1ull << s.tile_shift, round = tile * kRtQueues;
    uint64_t end = n / round * tile;  // positions of queue v below n, whole chunks
    const uint64_t rest = n % round;
    if (rest > v * tile) end += std::min<uint64_t>(tile, rest - v * tile);
    const uint64_t shared = rt_shared_out(s.blocks, wpb, s.share, v);
    end = std::max((end + s.chunk - 1) / s.chunk * s.chunk, shared);
    const uint64_t top = end + (uint64_t)waves * s.chunk;  // each wave adds a chunk once more than there is
    if (place(s.tile_shift, v, end) < n) bad("end of a queue", n, wg, max_blocks);
    if (top >= kRtQueuesDone || place(s.tile_shift, v, top) >> 32 ||
        place(s.tile_shift, v, top) != rt_ray_at(s.tile_shift, v, (uint32_t)top))
      bad("a head wraps", n, wg, max_blocks);
  }
}

int main() {
  std::mt19937 rng(7);
  long cases = 0;
  for (uint32_t wg : {64u, 128u, 256u})
    for (uint32_t blocks : {1u, 2u, 3u, 7u, 8u, 9u, 15u, 257u, 1280u, 2048u, 4095u})
      for (int k = 0; k < 14; ++k) {
        const uint64_t all = (uint64_t)blocks * wg;   // 64 rays on each wave
        const uint64_t edges[] = {1, 63, 64, 65, 1023, 1025, all - 1, all, all + 1, all + 65, all * 16, all * 16 + 1,
                                  all * 40 + 63, 1 + rng() % (all * 20)};
        const uint64_t n = edges[k];
        if (n < 1 || n > 0x7FFFFFFFull) continue;
        for (int order = 0; order < 3; ++order) hand_out((uint32_t)n, wg, blocks, order);
        ++cases;
      }
  for (int order = 0; order < 2; ++order) hand_out(0x7FFFFFFFu, 256, 1280, order);
  for (uint32_t wg : {64u, 128u, 256u})
    for (uint32_t blocks = 1; blocks <= 16384u * 256u / wg; ++blocks)
      for (uint32_t n : {0x7FFFFFFFu, 0x7FFFFFFFu - blocks, 0x40000001u}) heads(n, wg, blocks);
  std::printf("%ld cases, %d failures\n", cases, failures);
  return failures != 0;
}
"""


def test_every_ray_is_handed_out_once(tmp_path):
    """Shares and chunks of a launch cover every ray exactly once: for ragged
    counts, grids of less than eight workgroups, chunks above 64 rays and waves
    that stop at their range limit, whatever the order in which the waves come;
    and no queue head wraps at the largest launches."""
    run_driver(tmp_path, RAYS)


RESIDENT = r"""
#include <cstdio>
#include <initializer_list>
#include "rt_launch.h"
int main() {
  int failures = 0;
  // what fits, piece by piece
  for (uint32_t bytes = 1; bytes <= kLdsBytes; ++bytes) {
    uint32_t pieces = 0, fit = 0;
    while (pieces * kLdsPiece < bytes) ++pieces;
    while ((fit + 1) * pieces * kLdsPiece <= kLdsBytes) ++fit;
    if (rtk_lds_blocks(bytes) != fit) {
      std::printf("%u bytes: %u, %u fit\n", bytes, rtk_lds_blocks(bytes), fit);
      ++failures;
    }
  }
  // the stacks (and the sentinel entry) of every variant
  for (uint32_t wg : {64u, 128u, 256u})
    for (int stack : {8, 16, 32}) {
      const uint32_t bytes = (uint32_t)(rtk_lds_entries(stack, true, 4) + 1) * 8u * wg + 4u;
      if (rtk_lds_blocks(bytes) * (wg / 64u) < (uint32_t)kRtWavesPerCu) {
        std::printf("stack %d workgroup %u: %u waves\n", stack, wg, rtk_lds_blocks(bytes) * (wg / 64u));
        ++failures;
      }
      const uint32_t refs = (uint32_t)(rtk_lds_entries(stack, false, 4) + 1) * 4u * wg + 4u;
      if (rtk_lds_blocks(refs) * (wg / 64u) < (uint32_t)kRtWavesPerCu) {
        std::printf("any hit, stack %d workgroup %u: %u waves\n", stack, wg, rtk_lds_blocks(refs) * (wg / 64u));
        ++failures;
      }
      // the upper levels fill what is left, and no more
      for (int width : {4, 8}) {
        const uint32_t full = bytes + (uint32_t)rtk_top_nodes(width, (int)wg, (int)bytes) * 28u * (uint32_t)width;
        if (rtk_lds_blocks(full) * (wg / 64u) < (uint32_t)kRtWavesPerCu) {
          std::printf("stack %d workgroup %u width %d: %u bytes\n", stack, wg, width, full);
          ++failures;
        }
      }
    }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
"""


def test_resident_waves(tmp_path):
    """Workgroups that a CU's LDS holds, and the stacks of all variants at the
    number of waves that a launch is made for."""
    run_driver(tmp_path, RESIDENT)

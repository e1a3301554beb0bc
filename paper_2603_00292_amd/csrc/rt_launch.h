// rt_launch.h -- scratch of a traversal launch (librtq internal; host and
// device, no HIP).
#pragma once
#include <stddef.h>
#include <stdint.h>

// Ray queues of a launch (one per die of the chip) and the words between
// their heads (a cache line each).
constexpr uint32_t kRtQueues = 8, kRtQueueStride = 32;
constexpr uint32_t kRtCounterWords = kRtQueues * kRtQueueStride;

// LDS stack entries of a lane in the variant with `stack` entries: 4-byte
// references for any-hit and all-hit queries; closest hits keep an 8-byte
// (distance, reference) entry, and 5/8 as many, which holds eight workgroups
// of 256 threads in a CU's 160 KB.
constexpr int rtk_lds_entries(int stack, bool cull) { return cull ? stack * 5 / 8 : stack; }
constexpr bool rtk_stack_culls(bool any, int mode) { return !any && mode != 3; }
// global stack words per thread (4-byte references) for a bound of max_stack entries
constexpr size_t rtk_spill_words(uint32_t max_stack, uint32_t stack, bool any, int mode) {
  const uint32_t lds = (uint32_t)rtk_lds_entries((int)stack, rtk_stack_culls(any, mode));
  return max_stack > lds ? max_stack - lds : 1u;
}

// Scratch of rt_trace_closest_noalloc.  A launch is taken while the words
// below fit RT_NOALLOC_SCRATCH_BYTES: 64, two per refill_min rays, 256 per wave
// of a workgroup and a workgroup's stack entries past `stack`.  This is the
// published limit, not the use: a launch takes kRtCounterWords and
// rtk_spill_words for each thread of one workgroup or more.
constexpr size_t rtk_noalloc_budget(uint32_t n, uint32_t refill_min, uint32_t stack, uint32_t wg, uint32_t max_stack) {
  return 64 + 2 * ((size_t)n / refill_min + 1) + (wg / 64u) * 256u +
         (size_t)(max_stack > stack ? max_stack - stack : 1u) * wg;
}
// Words of the array behind it for a limit of `words`: closest hits keep 3/8
// of the variant's entries fewer in LDS, 12 for 32 entries, so that the
// deepest stack taken needs this much more (256 threads).
constexpr size_t rtk_noalloc_array(size_t words) {
  return words + kRtCounterWords + (32u - (uint32_t)rtk_lds_entries(32, true)) * 256u;
}

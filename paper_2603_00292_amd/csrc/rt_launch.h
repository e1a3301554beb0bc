// rt_launch.h -- grid, ray shares and scratch of a traversal launch (librtq
// internal; host and device, no HIP).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

// Ray queues of a launch (one per die of the chip) and the words between
// their heads (a cache line each).
constexpr uint32_t kRtQueues = 8, kRtQueueStride = 32;
constexpr uint32_t kRtCounterWords = kRtQueues * kRtQueueStride;
// set in a head once no queue has rays left (the positions stay below it)
constexpr uint32_t kRtQueuesDone = 0x80000000u;

// Closest queries on one accel (mode 0) finalize their hits inside the
// traversal kernel, each wave the ray ranges it took once they are all
// finished; a wave remembers at most this many ranges (one per lane) and then
// takes no more, so the chunks are sized for a quarter of that (launch_shape).
constexpr uint32_t kRtRangesPerWave = 64;

// Grid and ray shares of a launch.  chunk == 0: wave w of workgroup b takes
// `share` rays from rt_first_ray() on, and that is all of them.  Otherwise the
// rays are dealt in tiles of 1 << tile_shift to the queues in turn; the waves
// of workgroups q, q + kRtQueues, ... take the first shares of queue q (as long
// as a chunk), and from there on all waves take chunks of whichever queue.
struct LaunchShape {
  uint32_t blocks, share, chunk, tile_shift;
};

// Up to 64 rays per resident wave, every wave takes its rays at once, in one
// share, and the queues are not used.  Few rays are spread over the chip's
// 1,024 SIMDs first (64 rays on a 20,480-triangle mesh: 26 us a call with one
// ray a wave, 35 with 32), then 32 to a wave (65,536 rays: 49 us; 16 to a
// wave 58).  On either side of 64 the better way depends on the rays: one share
// a wave / queues, 250,007 rays on 1,310,720 triangles 211 / 237 us, on 1,024
// instances 227 / 228; 327,681 rays 229 / 226, instances 246 / 230, but 120 /
// 164 on 20,480 triangles; 500,009 rays 293 / 318, 295 / 301 and 129 / 143.  A
// long share can leave its costly rays to one wave, which queues do not.
// Beyond, waves take a chunk each and then more from the queues: 64
// rays, or more when the average wave would need more than a quarter of its
// kRtRangesPerWave ranges (the waves together can then hold four times the
// rays, so a wave with a full list always leaves the rest to others).  A queue
// gets at least 16 tiles, of at most 32,768 rays (tiles of 256 to 65,536 rays
// are within 3% of each other).
inline LaunchShape launch_shape(uint32_t n, uint32_t wg, uint32_t max_blocks) {
  LaunchShape s;
  const uint32_t wpb = wg / 64u;
  const uint64_t waves_max = (uint64_t)max_blocks * wpb;
  s.tile_shift = 0;
  if (n <= waves_max * 64u) {
    const uint32_t spread = std::min(32u, (n + 1023u) / 1024u);
    s.share = std::max(std::max(1u, spread), (uint32_t)((n + waves_max - 1) / waves_max));
    s.blocks = std::max(1u, (n + s.share * wpb - 1) / (s.share * wpb));
    s.chunk = 0;
  } else {
    s.blocks = max_blocks;
    s.chunk = 64;
    while ((uint64_t)s.chunk * (kRtRangesPerWave / 4u) * waves_max < n) s.chunk *= 2;
    s.share = s.chunk;
    while ((1u << s.tile_shift) < s.chunk ||
           (s.tile_shift < 15u && ((uint64_t)kRtQueues * 16u << (s.tile_shift + 1)) <= n))
      ++s.tile_shift;
  }
  return s;
}

// Place in the ray order of position p of queue v.  A queue's head runs past
// its rays by at most a chunk for each wave of the launch, and fewer than 2^31
// rays keep that below 2^32.
constexpr uint32_t rt_ray_at(uint32_t tile_shift, uint32_t v, uint32_t p) {
  return ((((p >> tile_shift) * kRtQueues) + v) << tile_shift) + (p & ((1u << tile_shift) - 1u));
}
// Rays of queue v that the first shares of `blocks` workgroups take.
constexpr uint32_t rt_shared_out(uint32_t blocks, uint32_t waves, uint32_t share, uint32_t v) {
  return (blocks + kRtQueues - 1u - v) / kRtQueues * waves * share;
}
// First ray of the share of wave `wave` of workgroup `block` (`waves` each).
constexpr uint32_t rt_first_ray(uint32_t block, uint32_t wave, uint32_t blocks, uint32_t waves, uint32_t share,
                                uint32_t chunk, uint32_t tile_shift) {
  const uint32_t v = block % kRtQueues, slot = block / kRtQueues;
  const uint32_t per = blocks / kRtQueues, rem = blocks % kRtQueues;
  return chunk == 0u ? ((v * per + (v < rem ? v : rem) + slot) * waves + wave) * share
                     : rt_ray_at(tile_shift, v, (slot * waves + wave) * share);
}

// LDS stack entries of a lane in the variant with `stack` entries: 4-byte
// references for any-hit and all-hit queries; closest hits keep 8-byte
// (distance, reference) entries, and as many as leave a CU's LDS to 20 waves:
// 8, 10 and 13.  (With 5 of the 8, 2-wide nodes spilled more than the cull
// saved: 400,003 incoherent rays 480 us against 437, workgroups of 64.)  Of 32
// references 16 lie in LDS where the upper tree levels can use the rest (any
// hit of 2,000,003 incoherent rays, workgroups of 256, 32 / 16: 4-wide nodes
// 580 / 512 us, 8-wide 700 / 585, but 2-wide, which have no such copy, 716 /
// 739).
constexpr int rtk_lds_entries(int stack, bool cull, int width) {
  return stack <= 8 ? stack : cull ? (stack <= 16 ? 10 : 13) : (width >= 4 ? 16 : stack);
}
constexpr bool rtk_stack_culls(bool any, int mode) { return !any && mode != 3; }
// global stack words per thread (4-byte references) for a bound of max_stack entries
constexpr size_t rtk_spill_words(uint32_t max_stack, uint32_t stack, bool any, int mode, int width) {
  const uint32_t lds = (uint32_t)rtk_lds_entries((int)stack, rtk_stack_culls(any, mode), width);
  return max_stack > lds ? max_stack - lds : 1u;
}

// A CU gives out its 160 KB of LDS in pieces of 1,280 bytes, which the runtime's
// occupancy query does not count: it named 15 workgroups of 64 threads and
// 10,756 bytes where 14 fit, and the last one then waited for a whole share of
// another (250,007 incoherent rays 383 us against 331 before the shares).
constexpr uint32_t kLdsBytes = 160 * 1024, kLdsPiece = 1280;
constexpr uint32_t rtk_lds_blocks(uint32_t bytes) {
  return bytes == 0u ? ~0u : kLdsBytes / ((bytes + kLdsPiece - 1u) / kLdsPiece * kLdsPiece);
}

// waves that run at once on a CU at most (see resident_blocks)
constexpr int kRtWavesPerCu = 20;

// Nodes of W-wide trees that fit the rest of a workgroup's LDS after `used`
// bytes, when kRtWavesPerCu waves are to share a CU's
constexpr int rtk_top_nodes(int width, int wg, int used) {
  const int budget = (int)(kLdsBytes / (kRtWavesPerCu * 64 / wg) / kLdsPiece * kLdsPiece) - 64;
  return budget > used ? (budget - used) / (28 * width) : 0;
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
// Words of the array behind it for a limit of `words`: closest hits keep fewer
// than the variant's entries in LDS, 19 fewer of 32, so that the deepest stack
// taken needs this much more (256 threads).
constexpr size_t rtk_noalloc_array(size_t words) {
  return words + kRtCounterWords + (32u - (uint32_t)rtk_lds_entries(32, true, 4)) * 256u;
}

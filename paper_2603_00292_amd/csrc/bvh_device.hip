// bvh_device.hip -- device-side BVH construction of one mesh (see bvh_device.h).
//
// Steps, each a kernel (or a hipCUB primitive) on the caller's stream:
//   1. compact float3 / uint3 copies of the strided mesh, index range check;
//   2. per triangle: validity (finite vertices, non-zero float64 normal),
//      the centre of its box, and the bounds of the valid centres;
//   3. compaction of the valid triangle ids (hipCUB select);
//   4. 30-bit Morton code of each centre within the bounds that step 2 left,
//      and a stable radix sort of (code, id) pairs (hipCUB);
//   5. bottom-up clustering (§6.2 construction paragraph: every triangle
//      starts as a cluster and clusters are merged until one is left) by
//      PLOC (Meister & Bittner 2018): the clusters stay in Morton order; each
//      finds, among the kPlocRadius clusters on either side, the one whose
//      merged box has the least surface area; mutual nearest neighbours are
//      merged into a new node; the list is compacted; repeat.  One pass is
//      two launches (pairs, merge + compaction), and
//      the passes below 1,024 clusters are one launch of one workgroup; new
//      nodes are numbered by position, so the tree is the same on every run;
//   6. the binary tree collapsed into W-wide nodes level by level (the
//      widest-child expansion of the host builder), leaves holding subtrees
//      of at most max_leaf triangles; each subtree gets a contiguous range of
//      triangle records, handed down from its parent;
//   7. triangle records in that order (vertices sorted, corner order kept).
#include "bvh_device.h"
#include "rt_alloc.h"

#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>

namespace rtd {
namespace {


// order-preserving map of a float to an unsigned int (for atomic min / max)
__device__ __forceinline__ uint32_t ord(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unord(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

__global__ void copy_vertices_kernel(const uint8_t* src, uint32_t stride, uint32_t n, float* dst) {
  uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  const float* p = reinterpret_cast<const float*>(src + (size_t)i * stride);
  dst[3 * (size_t)i + 0] = p[0];
  dst[3 * (size_t)i + 1] = p[1];
  dst[3 * (size_t)i + 2] = p[2];
}

__global__ void copy_indices_kernel(const uint8_t* src, uint32_t stride, uint32_t n,
                                    uint32_t vertex_count, uint32_t* dst, uint32_t* error) {
  uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  const uint32_t* p = reinterpret_cast<const uint32_t*>(src + (size_t)i * stride);
  uint32_t a = p[0], b = p[1], c = p[2];
  if (a >= vertex_count || b >= vertex_count || c >= vertex_count) atomicOr(error, 1u);
  dst[3 * (size_t)i + 0] = a;
  dst[3 * (size_t)i + 1] = b;
  dst[3 * (size_t)i + 2] = c;
}

__device__ __forceinline__ void load_tri(const float* V, const uint32_t* I, uint32_t t, float p[3][3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    uint32_t v = I[3 * (size_t)t + k];
#pragma unroll
    for (int a = 0; a < 3; ++a) p[k][a] = V[3 * (size_t)v + a];
  }
}

// Blocks of the first pass over the triangles, at most; each leaves the bounds
// of its valid centres in a row of its own, and the Morton kernel's blocks
// reduce the rows.  Atomics on six words from every 256 triangles took 90 us
// at 327,680 triangles; this takes no launch and adds 5 us to the pass.
constexpr uint32_t kPrepBlocks = 256;

// minimum (k < 3) and maximum (k >= 3) over the block; v valid in every thread
__device__ __forceinline__ void reduce_bounds(uint32_t (&v)[6], uint32_t (*s)[4]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    for (int o = 32; o > 0; o >>= 1) {
      const uint32_t x = (uint32_t)__shfl_xor((int)v[k], o);
      v[k] = k < 3 ? min(v[k], x) : max(v[k], x);
    }
    if ((threadIdx.x & 63u) == 0u) s[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 6; ++k)
#pragma unroll
    for (int w = 0; w < 4; ++w) v[k] = k < 3 ? min(v[k], s[k][w]) : max(v[k], s[k][w]);
}

// validity (indices in range, finite vertices, non-zero float64 normal), box
// centre, and the bounds of the valid centres: order-preserving codes, min
// x, y, z and max x, y, z, one row per block
__global__ __launch_bounds__(256) void prep_kernel(const float* V, const uint32_t* I, uint32_t n, uint32_t nv,
                                                   uint8_t* valid, float4* centre, uint32_t* bounds) {
  __shared__ uint32_t s[6][4];
  uint32_t v[6] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u, 0u};
  for (uint64_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
    if (I[3 * i] >= nv || I[3 * i + 1] >= nv || I[3 * i + 2] >= nv) {  // the build ends in an error
      valid[i] = 0;
      continue;
    }
    float p[3][3];
    load_tri(V, I, (uint32_t)i, p);
    bool finite = true;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int a = 0; a < 3; ++a) finite = finite && (fabsf(p[k][a]) < __int_as_float(0x7f800000));
    double e1x = (double)p[1][0] - p[0][0], e1y = (double)p[1][1] - p[0][1], e1z = (double)p[1][2] - p[0][2];
    double e2x = (double)p[2][0] - p[0][0], e2y = (double)p[2][1] - p[0][1], e2z = (double)p[2][2] - p[0][2];
    double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
    const bool ok = finite && !(nx == 0.0 && ny == 0.0 && nz == 0.0);
    valid[i] = ok ? 1 : 0;
    float c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float lo = fminf(fminf(p[0][a], p[1][a]), p[2][a]);
      float hi = fmaxf(fmaxf(p[0][a], p[1][a]), p[2][a]);
      c[a] = 0.5f * lo + 0.5f * hi;
      if (ok) {
        v[a] = min(v[a], ord(c[a]));
        v[3 + a] = max(v[3 + a], ord(c[a]));
      }
    }
    centre[i] = make_float4(c[0], c[1], c[2], 0.0f);
  }
  reduce_bounds(v, s);
  if (threadIdx.x == 0)
    for (int k = 0; k < 6; ++k) bounds[6 * blockIdx.x + k] = v[k];
}

__device__ __forceinline__ uint32_t spread10(uint32_t x) {
  x &= 0x3FFu;
  x = (x | (x << 16)) & 0x030000FFu;
  x = (x | (x << 8)) & 0x0300F00Fu;
  x = (x | (x << 4)) & 0x030C30C3u;
  x = (x | (x << 2)) & 0x09249249u;
  return x;
}

// 30-bit Morton code of each valid centre.  The sort is stable and the ids
// arrive in ascending order, so equal codes stay in order of their ids.
__global__ __launch_bounds__(256) void morton_kernel(const float4* centre, const uint32_t* ids, uint32_t m,
                                                     const uint32_t* bounds, uint32_t rows, uint32_t* keys) {
  __shared__ uint32_t s[6][4];
  uint32_t v[6] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u, 0u};
  if (threadIdx.x < rows)  // at most kPrepBlocks = 256
    for (int k = 0; k < 6; ++k) v[k] = bounds[6 * threadIdx.x + k];
  reduce_bounds(v, s);
  uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= m) return;
  float4 c = centre[ids[i]];
  float cc[3] = {c.x, c.y, c.z};
  uint32_t q[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float lo = unord(v[a]), hi = unord(v[3 + a]);
    float ext = hi - lo;
    float x = ext > 0.0f ? (cc[a] - lo) / ext * 1024.0f : 0.0f;
    x = fminf(fmaxf(x, 0.0f), 1023.0f);
    q[a] = (uint32_t)x;
  }
  keys[i] = spread10(q[0]) | (spread10(q[1]) << 1) | (spread10(q[2]) << 2);
}

// ---------------------------------------------------------------------------
// PLOC.  Binary node ids: leaf k (k-th triangle in Morton order) is m - 1 + k;
// internal nodes take ids m - 2, m - 3, ... in the order they are made, so
// the last merge makes the root, node 0.
// ---------------------------------------------------------------------------
// Search radius: on the 1.3M-triangle icosphere, radii 8 / 16 / 32 / 64 gave
// 20.6 / 21.3 / 20.4 / 20.8 node visits per incoherent ray; 32 is kept.
constexpr int kPlocRadius = 32;

// Where a pass stands: the n clusters are list `side`; `made` merges have
// been done; `force` is set after a pass without a mutual pair (possible only
// through exact ties of both area and hash), and then (2k, 2k + 1) are paired.
// Pass p reads entry p and writes entry p + 1, so the passes of a batch are
// launched without the host between them.
struct PlocState {
  uint32_t n, made, force, side;
};

__global__ void leaf_boxes_kernel(const float* V, const uint32_t* I, const uint32_t* sorted_ids, uint32_t m,
                                  float* box, uint32_t* count, uint32_t* clusters, PlocState* state) {
  uint32_t k = blockIdx.x * 256u + threadIdx.x;
  if (k >= m) return;
  if (k == 0u) state[0] = PlocState{m, 0u, 0u, 0u};
  float p[3][3];
  load_tri(V, I, sorted_ids[k], p);
  uint32_t id = m - 1u + k;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    box[6 * (size_t)id + a] = fminf(fminf(p[0][a], p[1][a]), p[2][a]);
    box[6 * (size_t)id + 3 + a] = fmaxf(fmaxf(p[0][a], p[1][a]), p[2][a]);
  }
  count[id] = 1u;
  clusters[k] = id;
}

// symmetric 32-bit hash of a pair of positions (a < b): breaks ties between
// equal merged areas so that duplicate boxes still pair up (multiplicative
// mixing followed by the MurmurHash3 finaliser)
__device__ __forceinline__ uint32_t pair_hash(uint32_t a, uint32_t b) {
  uint32_t h = a * 0x9E3779B1u + b * 0x85EBCA77u + 0x165667B1u;
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}

// A better neighbour by (area bits, pair hash, position): a pair's order is
// the same from either side, so mutual neighbours are well defined.  The hash
// is five quarter-rate multiplies and settles ties only, so it is computed
// only for those.
__device__ __forceinline__ uint32_t tie_hash(uint32_t i, uint32_t j) { return pair_hash(min(i, j), max(i, j)); }
__device__ __forceinline__ void ploc_take(uint32_t i, uint32_t j, uint32_t bits, uint32_t& best, uint32_t& arg) {
  if (bits == best && tie_hash(i, j) < tie_hash(i, arg)) arg = j;
  if (bits < best) {
    best = bits;
    arg = j;
  }
}

// Half surface area of the box around two boxes (rows of lo xyz, hi xyz), as
// bits: it is >= 0, because boxes are finite and not inverted.
template <int T>
__device__ __forceinline__ uint32_t merged_area(const float (&mine)[6], const float (*sb)[T], int l) {
  float dx = fmaxf(mine[3], sb[3][l]) - fminf(mine[0], sb[0][l]);
  float dy = fmaxf(mine[4], sb[4][l]) - fminf(mine[1], sb[1][l]);
  float dz = fmaxf(mine[5], sb[5][l]) - fminf(mine[2], sb[2][l]);
  return __float_as_uint(dx * dy + dy * dz + dz * dx);
}

// The best of `width` threads (a power of two, up to 64) that searched for i.
__device__ __forceinline__ void ploc_best(uint32_t i, uint32_t width, uint32_t& best, uint32_t& arg) {
  for (uint32_t o = 1u; o < width; o <<= 1) {
    const uint32_t b2 = __shfl_xor(best, (int)o), a2 = __shfl_xor(arg, (int)o);
    bool take = b2 < best;
    if (b2 == best && a2 != arg) {  // a thread without a candidate has the position itself
      const uint32_t h1 = tie_hash(i, arg), h2 = tie_hash(i, a2);
      take = h2 < h1 || (h2 == h1 && a2 < arg);
    }
    if (take) {
      best = b2;
      arg = a2;
    }
  }
}

struct PlocParams {
  PlocState* state;    // kPlocBatch + 1 entries
  uint32_t* list[2];   // cluster ids in Morton order
  uint32_t* partner;   // of each position in this pass: the other half of its pair, n if none
  uint2* sums;         // per tile of the pair kernel: lower and upper halves of pairs
  uint32_t *left, *right, *count;
  float* box;
  uint32_t m;
};

// The multi-block passes stop at kPlocTail clusters, where one workgroup
// finishes the tree out of LDS.  A pass is two launches of a few microseconds
// each whatever its size, and a pass of 1,024 clusters takes one compute unit
// about as long; below that it only gets cheaper (33 of the 55 passes over a
// 327,680-triangle mesh have 2,048 clusters or fewer).
constexpr uint32_t kPlocTail = 1024;
// Positions per workgroup of the merge kernel; a multiple of the pair
// kernel's tiles and even, so that the pairs of a forced pass stay in one.
constexpr uint32_t kPlocTile = 960;
constexpr uint32_t kPlocLarge = 1024 - 2 * kPlocRadius, kPlocSmall = 256 - 2 * kPlocRadius;
// A host synchronisation leaves the GPU idle for about 40 us, a pass that
// finds nothing left to do takes about 5 us.  A pass leaves about four fifths
// of its clusters (22 passes from 327,680 to 2,048), so as many passes are
// queued as that takes to reach kPlocTail; at least two, so that a pass without
// a pair and the forced one after it are in one batch and the count shrinks.
constexpr int kPlocBatch = 32;
constexpr float kPlocDecay = 0.23f;

// Sums of (lower, upper) over the block's threads before this one, and over
// all of them.  `part` is LDS for the block's waves; a barrier is passed
// before it is written and one after.
template <uint32_t WAVES>
__device__ __forceinline__ void pair_scan(bool lower, bool upper, uint2 (&part)[WAVES], uint2& before, uint2& all) {
  const uint64_t bl = __ballot(lower), bu = __ballot(upper);
  const uint64_t below = (1ull << (threadIdx.x & 63u)) - 1ull;
  const uint32_t wave = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63u) == 0u) part[wave] = make_uint2((uint32_t)__popcll(bl), (uint32_t)__popcll(bu));
  __syncthreads();
  before = make_uint2((uint32_t)__popcll(bl & below), (uint32_t)__popcll(bu & below));
  all = make_uint2(0u, 0u);
#pragma unroll
  for (uint32_t w = 0; w < WAVES; ++w) {
    const uint2 p = part[w];
    if (w < wave) {
      before.x += p.x;
      before.y += p.y;
    }
    all.x += p.x;
    all.y += p.y;
  }
}

// The partner of position i in this pass: its nearest neighbour when the
// relation is mutual (in a forced pass its even/odd partner); n if none.
// `nn` holds the neighbours of the positions from `first` on.
template <typename N>
__device__ __forceinline__ uint32_t ploc_partner(const N* nn, int first, uint32_t n, uint32_t force, uint32_t i) {
  if (force) {
    uint32_t j = i ^ 1u;
    return j < n ? j : n;
  }
  const uint32_t j = nn[(int)i - first];
  return (j != i && nn[(int)j - first] == i) ? j : n;
}

// The pairs of a pass.  The nearest neighbour of position i is the cluster
// among [i - r, i + r] whose merged box with i has the least half surface area
// (ties: the pair hash).  A tile of T - 2r positions also finds the neighbours
// of the r positions on either side, so that it settles its own pairs and
// counts them without another launch (3.8 us and a gap, and a pass over 20,000
// clusters took 12).  Large passes are bound by the searches: T = 1,024 makes
// 7% more of them.  Small ones are bound by the chain of 64 boxes a search, and
// the chip has threads to spare: T = 256, which makes a third more, and four
// threads a search (11.0 -> 7.3 us a pass).  All passes over a 327,680-triangle
// mesh, kernels only: 714 us with a launch for the neighbours and one to count
// the pairs, 550 us this way.
template <int T, int S>
__global__ __launch_bounds__(T * S) void ploc_pair_kernel(PlocParams P, int pass) {
  constexpr int R = kPlocRadius, kBoxes = T + 2 * R, kIn = T - 2 * R;
  static_assert(kPlocTile % kIn == 0 && kIn % 2 == 0, "tiles of the merge kernel");
  __shared__ float sb[6][kBoxes];
  __shared__ uint32_t nn[T];
  __shared__ uint2 part[T * S / 64];
  const PlocState st = P.state[pass];
  const int n = (int)st.n;
  const int first = (int)(blockIdx.x * (uint32_t)kIn);
  if (st.n <= kPlocTail || first >= n) return;
  if (!st.force) {
    const uint32_t* clusters = P.list[st.side];
    const int base = first - 2 * R;  // position of sb[.][0]
    for (int t = threadIdx.x; t < kBoxes; t += T * S) {
      const int i = base + t;
      if (i >= 0 && i < n) {
        const float* q = P.box + 6 * (size_t)clusters[i];
#pragma unroll
        for (int a = 0; a < 6; ++a) sb[a][t] = q[a];
      }
    }
    __syncthreads();
    const int i = first - R + (int)threadIdx.x / S;
    uint32_t best = 0xFFFFFFFFu, arg = (uint32_t)i;
    if (i >= 0 && i < n) {
      float mine[6];
#pragma unroll
      for (int a = 0; a < 6; ++a) mine[a] = sb[a][i - base];
      const int jlo = max(i - R, 0), jhi = min(i + R, n - 1);
#pragma unroll 4
      for (int j = jlo + (int)threadIdx.x % S; j <= jhi; j += S)
        if (j != i) ploc_take((uint32_t)i, (uint32_t)j, merged_area<kBoxes>(mine, sb, j - base), best, arg);
    }
    ploc_best((uint32_t)i, S, best, arg);
    if ((int)threadIdx.x % S == 0) nn[threadIdx.x / S] = arg;  // (positions outside the list are not read)
    __syncthreads();
  }
  const uint32_t i = (uint32_t)first + threadIdx.x;
  uint32_t j = st.n;
  if ((int)threadIdx.x < kIn && i < st.n) {
    j = ploc_partner(nn, first - R, st.n, st.force, i);
    P.partner[i] = j;
  }
  uint2 before, all;
  pair_scan(j < st.n && i < j, j < st.n && j < i, part, before, all);
  if (threadIdx.x == 0) P.sums[blockIdx.x] = all;
}

// The lower position of a merged pair makes node m - 2 - (merges before it)
// and keeps its place in the list; the upper one is dropped.  Every block adds
// up the sums of the tiles before its own (`per` of the pair kernel's to one
// of its own), which takes the place of a scan and a selection of their own.
// Those reads grow with the square of the tiles: a whole build took 4.6 ms at
// 4,000,000 triangles (with scan and selection 16.2), 12.8 at 16,000,000 (33.6)
// and 27.5 at 40,000,000 (67.5), so up to there they do not show.
__global__ __launch_bounds__(1024) void ploc_merge_kernel(PlocParams P, int pass, uint32_t per) {
  __shared__ uint2 part[16];
  __shared__ uint2 sum_before;
  const PlocState st = P.state[pass];
  if (st.n <= kPlocTail) {
    if (blockIdx.x == 0 && threadIdx.x == 0) P.state[pass + 1] = st;
    return;
  }
  if (blockIdx.x * kPlocTile >= st.n) return;
  if (threadIdx.x == 0) sum_before = make_uint2(0u, 0u);
  __syncthreads();
  uint2 own = make_uint2(0u, 0u);
  for (uint32_t b = threadIdx.x; b < blockIdx.x * per; b += 1024u) {
    const uint2 p = P.sums[b];
    own.x += p.x;
    own.y += p.y;
  }
  for (int o = 32; o > 0; o >>= 1) {
    own.x += __shfl_down(own.x, o);
    own.y += __shfl_down(own.y, o);
  }
  if ((threadIdx.x & 63u) == 0u && own.x + own.y != 0u) {
    atomicAdd(&sum_before.x, own.x);
    atomicAdd(&sum_before.y, own.y);
  }
  const uint32_t n = st.n, i = blockIdx.x * kPlocTile + threadIdx.x;
  const bool mine = threadIdx.x < kPlocTile && i < n;
  const uint32_t j = mine ? P.partner[i] : n;
  const bool lower = j < n && i < j, upper = j < n && j < i;
  uint2 before, all;
  pair_scan(lower, upper, part, before, all);  // its barriers order sum_before as well
  const uint2 tiles = sum_before;
  const uint32_t* in = P.list[st.side];
  uint32_t* out = P.list[st.side ^ 1u];
  if (mine && !upper) {
    const uint32_t ci = in[i];
    uint32_t id = ci;
    if (lower) {
      const uint32_t cj = in[j];
      id = P.m - 2u - st.made - (tiles.x + before.x);
      P.left[id] = ci;
      P.right[id] = cj;
      P.count[id] = P.count[ci] + P.count[cj];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        P.box[6 * (size_t)id + a] = fminf(P.box[6 * (size_t)ci + a], P.box[6 * (size_t)cj + a]);
        P.box[6 * (size_t)id + 3 + a] = fmaxf(P.box[6 * (size_t)ci + 3 + a], P.box[6 * (size_t)cj + 3 + a]);
      }
    }
    out[i - (tiles.y + before.y)] = id;
  }
  if (blockIdx.x == (n - 1u) / kPlocTile && threadIdx.x == 0) {
    const uint32_t pairs = tiles.x + all.x;
    P.state[pass + 1] = PlocState{n - pairs, st.made + pairs, pairs == 0u ? 1u : 0u, st.side ^ 1u};
  }
}

// The last passes, at most kPlocTail clusters, in one workgroup with the boxes
// in LDS.  Bound by the chain of passes: a search of 64 neighbours and four
// barriers each.  The search of one cluster is spread over as many threads as
// there are to spare (up to 32).
__global__ __launch_bounds__(1024) void ploc_tail_kernel(PlocParams P, int pass) {
  constexpr int T = (int)kPlocTail;
  __shared__ float sb[6][T];
  __shared__ uint32_t ids[T], cnt[T];
  __shared__ uint16_t nn[T];
  __shared__ uint2 part[16];
  PlocState st = P.state[pass];
  if (st.n > kPlocTail) {  // not there yet: the next batch goes on from entry 0
    if (threadIdx.x == 0) P.state[0] = st;
    return;
  }
  const uint32_t t = threadIdx.x;
  if (t < st.n) {
    const uint32_t c = P.list[st.side][t];
    ids[t] = c;
    cnt[t] = P.count[c];
#pragma unroll
    for (int a = 0; a < 6; ++a) sb[a][t] = P.box[6 * (size_t)c + a];
  }
  __syncthreads();
  while (st.n > 1u) {
    const uint32_t n = st.n;
    if (!st.force) {
      uint32_t s = 0;
      while (s < 5u && (n << (s + 1u)) <= 1024u) ++s;
      const uint32_t i = t >> s;
      uint32_t best = 0xFFFFFFFFu, arg = i;
      if (i < n) {
        float mine[6];
#pragma unroll
        for (int a = 0; a < 6; ++a) mine[a] = sb[a][i];
        const int lo = max((int)i - kPlocRadius, 0), hi = min((int)i + kPlocRadius, (int)n - 1);
#pragma unroll 4
        for (int j = lo + (int)(t & ((1u << s) - 1u)); j <= hi; j += 1 << s)
          if (j != (int)i) ploc_take(i, (uint32_t)j, merged_area<T>(mine, sb, j), best, arg);
      }
      ploc_best(i, 1u << s, best, arg);
      if (i < n && (t & ((1u << s) - 1u)) == 0u) nn[i] = (uint16_t)arg;
    }
    __syncthreads();
    const uint32_t j = t < n ? ploc_partner(nn, 0, n, st.force, t) : n;
    const bool lower = j < n && t < j, upper = j < n && j < t;
    uint32_t id = 0u, c = 0u;
    float q[6];
    uint2 before, all;
    pair_scan(lower, upper, part, before, all);
    if (t < n) {
      id = ids[t];
      c = cnt[t];
#pragma unroll
      for (int a = 0; a < 6; ++a) q[a] = sb[a][t];
      if (lower) {
        const uint32_t made = P.m - 2u - st.made - before.x;
        P.left[made] = id;
        P.right[made] = ids[j];
        c += cnt[j];
        P.count[made] = c;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          q[a] = fminf(q[a], sb[a][j]);
          q[3 + a] = fmaxf(q[3 + a], sb[3 + a][j]);
        }
#pragma unroll
        for (int a = 0; a < 6; ++a) P.box[6 * (size_t)made + a] = q[a];
        id = made;
      }
    }
    __syncthreads();
    if (t < n && !upper) {
      const uint32_t to = t - before.y;
      ids[to] = id;
      cnt[to] = c;
#pragma unroll
      for (int a = 0; a < 6; ++a) sb[a][to] = q[a];
    }
    st = PlocState{n - all.x, st.made + all.x, all.x == 0u ? 1u : 0u, 0u};
    __syncthreads();
  }
  if (t == 0) P.state[0] = st;
}

// A subtree waiting to become a wide node; the items are indexed by wide node.
struct Item {
  uint32_t bnode;   // binary node id
  uint32_t stack;   // stack entries above this node
  uint32_t first;   // first triangle record of the subtree
};

// A leaf waiting for its triangles to be listed.
struct LeafItem {
  uint32_t bnode;
  uint32_t first;
};

// Levels collapsed per host synchronisation (about 40 us of an idle GPU; a
// level with nothing in it takes about 3 us).
constexpr uint32_t kLevelBatch = 16;

struct CollapseState {
  uint32_t cnt[kLevelBatch + 1];  // wide nodes of each level of the batch
  uint32_t leaves;
  uint32_t max_stack;
  float root_box[6];
  double area;
};

struct CollapseParams {
  const uint32_t* left;
  const uint32_t* right;
  const uint32_t* count;   // triangles below each binary node
  const float* box;
  Item* items;
  LeafItem* leaf_items;
  CollapseState* state;
  float* nodes;
  uint32_t m;
  uint32_t max_leaf;
};

__device__ __forceinline__ double area_of(const float* q) {
  double dx = (double)q[3] - q[0], dy = (double)q[4] - q[1], dz = (double)q[5] - q[2];
  return 2.0 * (dx * dy + dy * dz + dz * dx);
}

// one thread: the state of the first batch (from_batch false; also the root
// item) or of the next one, whose first level is the last one's successor
__global__ void collapse_begin_kernel(CollapseParams P, bool from_batch) {
  CollapseState& st = *P.state;
  st.cnt[0] = from_batch ? st.cnt[kLevelBatch] : 1u;
  for (uint32_t l = 1; l <= kLevelBatch; ++l) st.cnt[l] = 0u;
  if (from_batch) return;
  st.leaves = 0u;
  st.max_stack = 0u;
  st.area = 0.0;
  for (int a = 0; a < 6; ++a) st.root_box[a] = P.box[a];
  P.items[0] = Item{0u, 0u, 0u};  // the binary root is internal node 0, or the only leaf when m == 1
}

// Level `level` of a batch whose first wide node is `base`: one wide node per
// thread by widest-child expansion.  Bound by its chain of dependent loads
// (four rounds of children, counts and boxes), so the children's boxes, sizes
// and areas stay in registers, listing a leaf's triangles is left to a kernel
// over all leaves at once, and a block takes its wide node numbers, its leaf
// slots and its part of the totals with one atomic each: 28 -> 9 us a level of
// a 327,680-triangle mesh.  A block's new nodes are numbered in order, so
// siblings lie next to each other.
template <int W>
__global__ __launch_bounds__(256) void collapse_kernel(CollapseParams P, uint32_t level, uint32_t base) {
  __shared__ uint32_t wave_big[4], wave_leaf[4], wave_stack[4];
  __shared__ double wave_area[4];
  __shared__ uint32_t at[2];
  uint32_t begin = base;
  for (uint32_t l = 0; l < level; ++l) begin += P.state->cnt[l];
  const uint32_t n_in = P.state->cnt[level];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  for (uint32_t t0 = blockIdx.x * 256u; t0 < n_in; t0 += gridDim.x * 256u) {
    const uint32_t t = t0 + threadIdx.x;
    const bool on = t < n_in;
    uint32_t kid[W], cnt[W];
    float box[W][6];
    double area[W];  // of children that are still to be split; -1 for the others
    uint32_t nk = 0, big = 0, leaf = 0, first = 0, stack_here = 0;
    double own_area = 0.0;
    if (on) {
      const Item it = P.items[begin + t];
      first = it.first;
      auto load = [&](uint32_t b, uint32_t& k, uint32_t& c, float (&q)[6], double& a) {
        k = b;
        c = P.count[b];
#pragma unroll
        for (int x = 0; x < 6; ++x) q[x] = P.box[6 * (size_t)b + x];
        a = b < P.m - 1u && c > P.max_leaf ? area_of(q) : -1.0;
      };
      load(it.bnode, kid[0], cnt[0], box[0], area[0]);
      own_area = area_of(box[0]);
      nk = 1;
#pragma unroll
      for (int step = 1; step < W; ++step) {
        int pick = -1;
        double best = -1.0;
#pragma unroll
        for (int i = 0; i < step; ++i)
          if ((uint32_t)i < nk && area[i] > best) {
            best = area[i];
            pick = i;
          }
        if (pick < 0) break;
        uint32_t b = 0;
#pragma unroll
        for (int i = 0; i < step; ++i)
          if (i == pick) b = kid[i];
        const uint32_t bl = P.left[b], br = P.right[b];
        uint32_t lk, lc, rk, rc;
        float lq[6], rq[6];
        double la, ra;
        load(bl, lk, lc, lq, la);
        load(br, rk, rc, rq, ra);
#pragma unroll
        for (int i = step; i >= 0; --i) {  // children after the split one move up
          if (i > pick + 1 && i > 0) {
            kid[i] = kid[i - 1];
            cnt[i] = cnt[i - 1];
            area[i] = area[i - 1];
#pragma unroll
            for (int x = 0; x < 6; ++x) box[i][x] = box[i - 1][x];
          } else if (i == pick + 1) {
            kid[i] = rk;
            cnt[i] = rc;
            area[i] = ra;
#pragma unroll
            for (int x = 0; x < 6; ++x) box[i][x] = rq[x];
          } else if (i == pick) {
            kid[i] = lk;
            cnt[i] = lc;
            area[i] = la;
#pragma unroll
            for (int x = 0; x < 6; ++x) box[i][x] = lq[x];
          }
        }
        ++nk;
      }
      stack_here = it.stack + nk - 1u;
#pragma unroll
      for (int i = 0; i < W; ++i)
        if ((uint32_t)i < nk) {
          if (area[i] >= 0.0) ++big;
          else ++leaf;
        }
    }
    // numbers before this thread in the block, and the block's totals
    uint32_t big_at = big, leaf_at = leaf, top = on ? stack_here + 1u : 0u;
    for (uint32_t o = 1; o < 64u; o <<= 1) {
      const uint32_t b2 = __shfl_up(big_at, o), l2 = __shfl_up(leaf_at, o);
      if (lane >= o) {
        big_at += b2;
        leaf_at += l2;
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      top = max(top, (uint32_t)__shfl_xor((int)top, o));
      own_area += __shfl_xor(own_area, o);
    }
    __syncthreads();
    if (lane == 63u) {
      wave_big[wave] = big_at;
      wave_leaf[wave] = leaf_at;
      wave_stack[wave] = top;
      wave_area[wave] = own_area;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t b = 0, l = 0, s = 0;
      double a = 0.0;
      for (int w = 0; w < 4; ++w) {
        b += wave_big[w];
        l += wave_leaf[w];
        s = max(s, wave_stack[w]);
        a += wave_area[w];
      }
      at[0] = b ? atomicAdd(&P.state->cnt[level + 1], b) : 0u;
      at[1] = l ? atomicAdd(&P.state->leaves, l) : 0u;
      atomicMax(&P.state->max_stack, s);
      atomicAdd(&P.state->area, a);
    }
    __syncthreads();
    uint32_t wide = begin + n_in + at[0] + big_at - big, slot = at[1] + leaf_at - leaf;
    for (uint32_t w = 0; w < wave; ++w) {
      wide += wave_big[w];
      slot += wave_leaf[w];
    }
    if (on) {
      float out[8][W];
#pragma unroll
      for (int i = 0; i < W; ++i) {
        uint32_t ref = RT_CHILD_EMPTY;
        const bool used = (uint32_t)i < nk;
        if (used) {
          if (area[i] >= 0.0) {
            P.items[wide] = Item{kid[i], stack_here, first};
            ref = wide++;
          } else {
            P.leaf_items[slot++] = LeafItem{kid[i], first};
            ref = RT_LEAF_BIT | (cnt[i] << RT_LEAF_COUNT_SHIFT) | first;
          }
          first += cnt[i];  // the children split the parent's record range in order
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          out[2 * a][i] = used ? box[i][a] : __int_as_float(0x7f800000);
          out[2 * a + 1][i] = used ? box[i][3 + a] : __int_as_float(0xff800000);
        }
        out[6][i] = __uint_as_float(ref);
        out[7][i] = 0.0f;
      }
      float* nd = P.nodes + (size_t)(begin + t) * 8 * W;
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int i = 0; i < W; ++i) nd[r * W + i] = out[r][i];
    }
  }
}

// the triangles of a leaf (at most max_leaf <= 15), depth first
__global__ void leaf_lists_kernel(CollapseParams P, uint32_t leaves, uint32_t* perm) {
  uint32_t t = blockIdx.x * 256u + threadIdx.x;
  if (t >= leaves) return;
  const LeafItem it = P.leaf_items[t];
  uint32_t stk[16];
  int sp = 0;
  uint32_t pos = it.first;
  stk[sp++] = it.bnode;
  while (sp > 0) {
    uint32_t x = stk[--sp];
    if (x >= P.m - 1u) {
      perm[pos++] = x - (P.m - 1u);
    } else {
      stk[sp++] = P.right[x];
      stk[sp++] = P.left[x];
    }
  }
}

__device__ __forceinline__ bool lex_less(const float* a, const float* b) {
  if (a[0] != b[0]) return a[0] < b[0];
  if (a[1] != b[1]) return a[1] < b[1];
  return a[2] < b[2];
}

// triangle record k = the triangle at Morton position perm[k]
__global__ void records_kernel(const float* V, const uint32_t* I, const uint32_t* sorted_ids,
                               const uint32_t* perm, uint32_t m, rt_tri_rec* out) {
  uint32_t k = blockIdx.x * 256u + threadIdx.x;
  if (k >= m) return;
  uint32_t prim = sorted_ids[perm[k]];
  float p[3][3];
  load_tri(V, I, prim, p);
  uint32_t corner[3] = {0u, 1u, 2u};
  auto cswap = [&](int a, int b) {
    if (lex_less(p[b], p[a])) {
      for (int c = 0; c < 3; ++c) {
        float t = p[a][c];
        p[a][c] = p[b][c];
        p[b][c] = t;
      }
      uint32_t t = corner[a];
      corner[a] = corner[b];
      corner[b] = t;
    }
  };
  cswap(0, 1);
  cswap(1, 2);
  cswap(0, 1);
  rt_tri_rec r;
  r.p0x = p[0][0]; r.p0y = p[0][1]; r.p0z = p[0][2];
  r.prim = prim;
  r.p1x = p[1][0]; r.p1y = p[1][1]; r.p1z = p[1][2];
  r.order = (0u << (2 * corner[0])) | (1u << (2 * corner[1])) | (2u << (2 * corner[2]));
  r.p2x = p[2][0]; r.p2y = p[2][1]; r.p2z = p[2][2];
  r.pad2 = 0;
  out[k] = r;
}

__global__ void relocate_kernel(float* nodes, uint32_t count, int W, uint32_t nb, uint32_t tb) {
  uint32_t t = blockIdx.x * 256u + threadIdx.x;
  if (t >= count * (uint32_t)W) return;
  uint32_t i = t / (uint32_t)W, c = t % (uint32_t)W;
  float* slot = nodes + (size_t)i * 8 * W + 6 * W + c;
  uint32_t ref = __float_as_uint(*slot);
  if (ref == RT_CHILD_EMPTY) return;
  if ((ref & RT_LEAF_BIT) == 0u) ref += nb;
  else if ((ref & RT_INST_BIT) == 0u) ref += tb;  // the first record is the low bits
  *slot = __uint_as_float(ref);
}

__global__ void fill_kernel(uint32_t* p, uint32_t n, uint32_t v) {
  uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) p[i] = v;
}

// n - 1 ... 0: wide nodes are numbered level by level, so this is deepest first
__global__ void reverse_kernel(uint32_t* p, uint32_t n) {
  uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) p[i] = n - 1u - i;
}

uint32_t blocks(uint64_t n) { return (uint32_t)((n + 255) / 256); }

// Arrays that share one allocation: each is asked for with want(), and
// commit() allocates them all and fills in the pointers.  A hipMalloc takes
// about 30 us and a hipFree, which waits for the device, about 80 us; one of
// each for every array was 2.1 of the 3.7 ms of a 327,680-triangle build and
// 5.0 of the 7.6 ms of a 1,310,720-triangle one.
struct Block {
  void* base = nullptr;
  size_t bytes = 0;
  std::vector<std::pair<void**, size_t>> slots;
  template <typename T>
  void want(T** p, size_t count) {
    slots.emplace_back(reinterpret_cast<void**>(p), bytes);
    bytes += (std::max<size_t>(count, 1) * sizeof(T) + 255) & ~(size_t)255;
  }
  hipError_t commit() {
    hipError_t e = rt_malloc(&base, bytes);
    if (e != hipSuccess) return e;
    for (auto& q : slots) *q.first = static_cast<char*>(base) + q.second;
    return hipSuccess;
  }
};

// temporaries, freed on every exit
struct Temps : Block {
  ~Temps() {
    if (base) (void)hipFree(base);
  }
};

template <typename T>
hipError_t keep(Output& out, T** p, size_t count) {
  *p = nullptr;
  if (count == 0) count = 1;
  hipError_t e = rt_malloc(reinterpret_cast<void**>(p), count * sizeof(T));
  if (e == hipSuccess) {
    out.owned.push_back(*p);
    out.owned_bytes += count * sizeof(T);
  }
  return e;
}

#define RTD_TRY(x)                     \
  do {                                 \
    hipError_t e_ = (x);               \
    if (e_ != hipSuccess) return e_;   \
  } while (0)

}  // namespace

hipError_t build(const Input& in, Output& out, bool& index_error, hipStream_t s) {
  index_error = false;
  const uint32_t nv = in.vertex_count, nt = in.triangle_count;
  const int W = in.width;
  // 1. compact copies and the index check
  RTD_TRY(keep(out, &out.vertices, (size_t)nv * 3));
  RTD_TRY(keep(out, &out.indices, (size_t)nt * 3));
  Temps tri_tmp;  // one row per input triangle
  uint32_t *err = nullptr, *ids = nullptr, *bounds = nullptr;
  uint8_t *valid = nullptr, *scratch = nullptr;
  float4* centre = nullptr;
  const uint32_t prep_blocks = std::min(std::max(blocks(nt), 1u), kPrepBlocks);
  hipcub::CountingInputIterator<uint32_t> counting(0);
  size_t bytes = 0;
  if (nt) RTD_TRY(hipcub::DeviceSelect::Flagged(nullptr, bytes, counting, valid, ids, err, (int)nt, s));
  tri_tmp.want(&err, 2);  // index error, valid triangles
  tri_tmp.want(&valid, nt);
  tri_tmp.want(&centre, nt);
  tri_tmp.want(&bounds, 6 * (size_t)prep_blocks);
  tri_tmp.want(&ids, nt);
  tri_tmp.want(&scratch, bytes);
  RTD_TRY(tri_tmp.commit());
  hipLaunchKernelGGL(fill_kernel, dim3(1), dim3(256), 0, s, err, 2u, 0u);
  if (nv) hipLaunchKernelGGL(copy_vertices_kernel, dim3(blocks(nv)), dim3(256), 0, s,
                             reinterpret_cast<const uint8_t*>(in.vertices), in.vertex_stride, nv, out.vertices);
  if (nt) hipLaunchKernelGGL(copy_indices_kernel, dim3(blocks(nt)), dim3(256), 0, s,
                             reinterpret_cast<const uint8_t*>(in.indices), in.index_stride, nt, nv, out.indices, err);
  RTD_TRY(hipGetLastError());
  // 2., 3. validity, centres and their bounds; valid ids
  out.refit_levels.assign(1, 0);
  if (nt) {
    hipLaunchKernelGGL(prep_kernel, dim3(prep_blocks), dim3(256), 0, s, out.vertices, out.indices, nt, nv, valid,
                       centre, bounds);
    RTD_TRY(hipGetLastError());
    RTD_TRY(hipcub::DeviceSelect::Flagged(scratch, bytes, counting, valid, ids, err + 1, (int)nt, s));
  }
  uint32_t h_err[2] = {0u, 0u};
  RTD_TRY(hipMemcpyAsync(h_err, err, sizeof(h_err), hipMemcpyDeviceToHost, s));
  RTD_TRY(hipStreamSynchronize(s));
  if (h_err[0]) {
    index_error = true;
    return hipSuccess;
  }
  const uint32_t m = h_err[1];
  out.tri_count = m;
  if (m == 0) return hipSuccess;
  // 4. Morton codes and the sort
  Temps tmp;  // rows per valid triangle, node or tile
  const uint32_t nb = 2 * m - 1;
  const size_t fpn = 8 * (size_t)W;
  uint32_t *keys = nullptr, *keys_sorted = nullptr, *ids_sorted = nullptr;
  uint8_t* sort_tmp = nullptr;
  uint32_t *left = nullptr, *right = nullptr, *count = nullptr, *perm = nullptr;
  uint32_t *cl_a = nullptr, *cl_b = nullptr, *partner = nullptr;
  uint2* sums = nullptr;
  PlocState* state = nullptr;
  float* box = nullptr;
  CollapseParams P{};
  bytes = 0;
  RTD_TRY(hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, keys, keys_sorted, ids, ids_sorted, (int)m, 0, 30, s));
  tmp.want(&keys, m);
  tmp.want(&keys_sorted, m);
  tmp.want(&ids_sorted, m);
  tmp.want(&sort_tmp, bytes);
  tmp.want(&left, m);
  tmp.want(&right, m);
  tmp.want(&count, nb);
  tmp.want(&perm, m);
  tmp.want(&cl_a, m);
  tmp.want(&cl_b, m);
  tmp.want(&partner, m);
  tmp.want(&sums, (m + kPlocSmall - 1) / kPlocSmall);
  tmp.want(&state, kPlocBatch + 1);
  tmp.want(&box, (size_t)nb * 6);
  tmp.want(&P.nodes, (size_t)m * fpn);  // at most m wide nodes
  tmp.want(&P.items, m);
  tmp.want(&P.leaf_items, m);
  tmp.want(&P.state, 1);
  RTD_TRY(tmp.commit());
  hipLaunchKernelGGL(morton_kernel, dim3(blocks(m)), dim3(256), 0, s, centre, ids, m, bounds, prep_blocks, keys);
  RTD_TRY(hipcub::DeviceRadixSort::SortPairs(sort_tmp, bytes, keys, keys_sorted, ids, ids_sorted, (int)m, 0, 30, s));
  // 5. PLOC
  hipLaunchKernelGGL(leaf_boxes_kernel, dim3(blocks(m)), dim3(256), 0, s, out.vertices, out.indices, ids_sorted, m,
                     box, count, cl_a, state);
  RTD_TRY(hipGetLastError());
  const PlocParams ploc{state, {cl_a, cl_b}, partner, sums, left, right, count, box, m};
  for (PlocState st{m, 0u, 0u, 0u};;) {
    const uint32_t tiles = (st.n + kPlocTile - 1) / kPlocTile;
    const float to_tail = std::log((float)st.n / (float)kPlocTail) / kPlocDecay;
    const int passes = st.n > kPlocTail ? std::min(std::max((int)std::ceil(to_tail), 2), kPlocBatch) : 0;
    for (int p = 0; p < passes; ++p) {
      // (the kernels take any number of clusters; this one is by the number
      // expected)
      const bool large = (float)st.n * std::exp(-kPlocDecay * (float)p) > 65536.0f;
      const uint32_t tile = large ? kPlocLarge : kPlocSmall;
      const dim3 pair_grid((st.n + tile - 1) / tile);
      if (large) hipLaunchKernelGGL((ploc_pair_kernel<1024, 1>), pair_grid, dim3(1024), 0, s, ploc, p);
      else hipLaunchKernelGGL((ploc_pair_kernel<256, 4>), pair_grid, dim3(1024), 0, s, ploc, p);
      hipLaunchKernelGGL(ploc_merge_kernel, dim3(tiles), dim3(1024), 0, s, ploc, p, kPlocTile / tile);
    }
    hipLaunchKernelGGL(ploc_tail_kernel, dim3(1), dim3(1024), 0, s, ploc, passes);
    RTD_TRY(hipGetLastError());
    const uint32_t n_old = st.n;
    RTD_TRY(hipMemcpyAsync(&st, state, sizeof(st), hipMemcpyDeviceToHost, s));
    RTD_TRY(hipStreamSynchronize(s));
    if (st.n == 1 && st.made == m - 1) break;  // m - 1 merges made ids m - 2 .. 0
    // cannot happen: a pass merges, or else the forced pass after it does
    if (st.n <= kPlocTail || st.n >= n_old) return hipErrorUnknown;
  }
  // 6. collapse, level by level; wide nodes of one level are numbered
  // consecutively, so the levels are index ranges
  P.left = left;
  P.right = right;
  P.count = count;
  P.box = box;
  P.m = m;
  P.max_leaf = (uint32_t)in.max_leaf;
  std::vector<uint32_t> level_begin{0u};
  CollapseState st{};
  const uint32_t level_blocks = std::min(blocks(m), 1024u);
  do {
    const uint32_t base = level_begin.back();
    hipLaunchKernelGGL(collapse_begin_kernel, dim3(1), dim3(1), 0, s, P, base != 0u);
    for (uint32_t l = 0; l < kLevelBatch; ++l) {
      if (W == 2) hipLaunchKernelGGL(collapse_kernel<2>, dim3(level_blocks), dim3(256), 0, s, P, l, base);
      else if (W == 4) hipLaunchKernelGGL(collapse_kernel<4>, dim3(level_blocks), dim3(256), 0, s, P, l, base);
      else hipLaunchKernelGGL(collapse_kernel<8>, dim3(level_blocks), dim3(256), 0, s, P, l, base);
    }
    RTD_TRY(hipGetLastError());
    RTD_TRY(hipMemcpyAsync(&st, P.state, sizeof(st), hipMemcpyDeviceToHost, s));
    RTD_TRY(hipStreamSynchronize(s));
    for (uint32_t l = 0; l < kLevelBatch && st.cnt[l] != 0u; ++l) level_begin.push_back(level_begin.back() + st.cnt[l]);
  } while (st.cnt[kLevelBatch] != 0u);
  // 7. triangle records in the order the collapse gave them
  const uint32_t node_count = level_begin.back();
  Block kept;
  kept.want(&out.nodes, (size_t)node_count * fpn);
  kept.want(&out.tris, m);
  kept.want(&out.refit_nodes, node_count);
  RTD_TRY(kept.commit());
  out.owned.push_back(kept.base);
  out.owned_bytes += (size_t)node_count * (fpn + 1) * 4 + (size_t)m * sizeof(rt_tri_rec);
  hipLaunchKernelGGL(leaf_lists_kernel, dim3(blocks(st.leaves)), dim3(256), 0, s, P, st.leaves, perm);
  hipLaunchKernelGGL(records_kernel, dim3(blocks(m)), dim3(256), 0, s, out.vertices, out.indices, ids_sorted, perm, m,
                     out.tris);
  RTD_TRY(hipGetLastError());
  // level_begin[l] .. level_begin[l+1] are the wide nodes of depth l+1
  out.node_count = node_count;
  for (int a = 0; a < 6; ++a) out.bounds[a] = st.root_box[a];
  out.leaf_count = st.leaves;
  out.max_stack = std::max(st.max_stack, 1u);
  out.max_depth = (uint32_t)level_begin.size() - 1;
  out.root = 0;
  double dx = (double)st.root_box[3] - st.root_box[0], dy = (double)st.root_box[4] - st.root_box[1],
         dz = (double)st.root_box[5] - st.root_box[2];
  double ra = 2.0 * (dx * dy + dy * dz + dz * dx);
  out.sah_cost = ra > 0.0 ? st.area / ra : 0.0;
  RTD_TRY(hipMemcpyAsync(out.nodes, P.nodes, (size_t)node_count * fpn * sizeof(float), hipMemcpyDeviceToDevice, s));
  // refit order: deepest level first
  hipLaunchKernelGGL(reverse_kernel, dim3(blocks(node_count)), dim3(256), 0, s, out.refit_nodes, node_count);
  for (size_t l = level_begin.size() - 1; l-- > 0;) out.refit_levels.push_back(node_count - level_begin[l]);
  RTD_TRY(hipGetLastError());
  RTD_TRY(hipStreamSynchronize(s));
  return hipSuccess;
}

hipError_t relocate(float* nodes, uint32_t node_count, int width, uint32_t node_base, uint32_t tri_base,
                    hipStream_t s) {
  if (node_count == 0) return hipSuccess;
  hipLaunchKernelGGL(relocate_kernel, dim3(blocks((uint64_t)node_count * width)), dim3(256), 0, s, nodes, node_count,
                     width, node_base, tri_base);
  return hipGetLastError();
}

}  // namespace rtd

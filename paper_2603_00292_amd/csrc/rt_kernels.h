// rt_kernels.h -- kernel parameter blocks and launch entry points of librtq
// (internal to the library; not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/rt.h"
#include "accumulate.h"
#include "rt_launch.h"
#include "rt_layout.h"

// One batch entry of a batched plan (device copy).
struct BatchDesc {
  const float* nodes;
  const rt_tri_rec* tris;
  const rt_mesh_dev* meshes;
  const rt_ray* rays;
  rt_hit* hits;
  uint32_t root;
  uint32_t count;
  const rt_inst_rec* insts;      // two-level plans
  const rt_inst_rec64* insts64;  // two-level plans
  uint32_t* inst_ids;            // two-level plans: instance ids out (may be null)
};

struct TraceParams {
  const float* nodes;
  const rt_tri_rec* tris;
  const rt_inst_rec* insts;
  const rt_inst_rec64* insts64;
  const rt_mesh_dev* meshes;
  const rt_ray* rays;
  rt_hit* hits;
  uint32_t* inst_ids;
  uint8_t* occluded;
  // See LaunchShape; counter[v * kRtQueueStride] counts the rays of queue v's
  // chunks given out, and carries kRtQueuesDone.  Zero before the launch, which
  // zeroes the heads at `clear` (NULL: none) for another one.
  uint32_t* counter;
  uint32_t* clear;
  uint32_t share, chunk, tile_shift;
  uint32_t* gstack;      // global stack: per thread of the grid, the entries past the LDS ones
  const BatchDesc* batches;
  const uint32_t* batch_offsets;  // batch_count + 1 prefix sums of counts
  uint32_t batch_count;
  uint32_t top_nodes;    // nodes [0, top_nodes) may be copied to LDS (upper levels first)
  uint32_t root;
  uint32_t n;            // rays in the launch (batched: total)
  uint32_t max_stack;    // stack entries a lane may need
  uint32_t gstride;      // threads in the grid
  uint32_t refill_min;   // refill a wave once this many lanes are idle
  uint64_t* counters;    // counting variants: node visits, triangle tests, spills
  uint32_t phase_counters;  // counting variants: also the wave-level loop counts (counters[4..7])
                         // (sums) and the deepest stack fill (maximum)
  uint32_t* status;      // host-mapped word: a lane of a counting variant
                         // sets it to 1 when a push would exceed max_stack
  // query options (modes 2 and 3; each may be null)
  const uint32_t* ray_masks;
  const uint32_t* skip_inst;
  const uint32_t* skip_prim;
  uint32_t* counts;      // mode 3: hits per ray
  uint32_t cap;          // mode 3: list entries per ray
};

// Single-level adjoint (a workgroup of 1024 threads per tile of rta::kTile
// rays): writes the ray gradients and places each hit ray's record in its
// bucket for the vertex accumulation of accumulate.h.
struct BackwardParams {
  rt_mesh_dev mesh;
  const float* tri_vertices;   // 9 floats per triangle: its vertices in index order
  const rt_ray* rays;
  const rt_hit* hits;
  const float* d_tuv;
  uint32_t n;
  float* d_origins;
  float* d_directions;
  rta::Bucketing bk;
};

// Adjoint of two-level closest hits (one thread per ray, two phases as
// above).  Vertex rows: vertex_base[mesh] + vertex id; frame rows:
// frame_row0 + 4 * instance + part, parts holding (S xyz), (q xyz),
// (q w, T x, T y), (T z, -, -).
struct BackwardInstParams {
  const rt_mesh_dev* meshes;      // device mesh records (the accel's copies)
  const uint64_t* vertex_base;    // first gradient row of each mesh
  const rt_inst_rec* insts;       // mesh of each instance
  const rt_inst_rec64* insts64;   // float64 world-to-object maps
  const rt_srt* srts;             // frames as given to the build
  uint32_t inst_count;
  const rt_ray* rays;
  const rt_hit* hits;
  const uint32_t* inst_ids;
  const float* d_tuv;
  uint32_t n;
  float* d_origins;
  float* d_directions;
  rta::Acc acc;
  uint32_t want_vertices;         // add vertex rows
  uint32_t want_frames;           // add frame rows
  uint32_t frame_row0;
  // bucketed form (backward_inst_tile_kernel): global-triangle vertex copy,
  // each instance's (first global triangle, triangle count), placements
  const float* tri_vertices;
  const uint2* inst_tris;
  rta::Bucketing vb, fb;
};

// Ambient-occlusion rays from closest hits (one thread per ray sample).
struct AoParams {
  rt_mesh_dev mesh;       // single level
  const rt_mesh_dev* meshes;  // two-level (device): every mesh
  const rt_inst_rec* insts;   // two-level: instance records (mesh id)
  const rt_srt* srts;         // two-level: frames
  const uint32_t* inst_ids;   // two-level: instance of each hit; null for single level
  uint32_t inst_count;
  const rt_ray* rays;
  const rt_hit* hits;
  const float* xi;        // n * samples * 2 uniforms
  rt_ray* out;            // n * samples rays
  uint32_t n;
  uint32_t samples;
  double offset;
  float radius;
  uint32_t block;        // samples of a workgroup (set by the launch)
};

// Kernel handle for a variant (mode 0: one accel, mode 1: batched closest,
// mode 2: one accel with query options, mode 3: all hits with query options;
// modes 2 and 3 exist for stack 16 / workgroup 256 only); nullptr when the
// combination is not compiled.  wide (stack 16 / workgroup 256 only): for
// accels whose node array does not fit 32-bit byte offsets; batched plans
// always use 64-bit addresses.
const void* rtk_trace_kernel(int width, int stack, int wg, bool any, bool inst, int mode, bool wide);
const void* rtk_count_kernel(int width, bool any, bool inst);
// Zeroes the queue heads of a launch to come on `stream` (a kernel: it may be
// captured).
hipError_t rtk_launch_queue_reset(uint32_t* counter, hipStream_t stream);
hipError_t rtk_launch_trace(const void* kern, uint32_t grid, uint32_t wg, const TraceParams& p,
                            hipStream_t stream);
// float64 finalize of closest hits written by a trace launch with the same params
hipError_t rtk_launch_finalize(bool inst, int mode, const TraceParams& p, hipStream_t stream);
// true when the traversal kernel of (any, inst, mode) finalizes its own hits
bool rtk_trace_fuses_finalize(bool any, bool inst, int mode);
// float64 finalize of the hit lists of an all-hits launch (n * cap entries)
hipError_t rtk_launch_finalize_all(bool inst, const TraceParams& p, hipStream_t stream);
hipError_t rtk_launch_backward(const BackwardParams& p, hipStream_t stream);
hipError_t rtk_launch_backward_inst(const BackwardInstParams& p, int phase, hipStream_t stream);
// the bucketed two-level adjoint (p.vb / p.fb placements; grid of kTile-ray tiles)
hipError_t rtk_launch_backward_inst_tiles(const BackwardInstParams& p, hipStream_t stream);
hipError_t rtk_launch_refit_tris(rt_tri_rec* tris, uint32_t n, const rt_mesh_dev& mesh,
                                 hipStream_t stream);
hipError_t rtk_launch_refit_nodes(int width, float* nodes, const rt_tri_rec* tris,
                                  const uint32_t* node_ids, uint32_t count, hipStream_t stream);
hipError_t rtk_launch_ao_rays(const AoParams& p, hipStream_t stream);
hipError_t rtk_launch_ao_resolve(const uint8_t* occluded, uint32_t n, uint32_t samples, float* ao,
                                 hipStream_t stream);

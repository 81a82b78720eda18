// gjp_internal.h -- host-side structures shared by the C ABI and the kernel
// launchers. Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>
#include <string>
#include <vector>

#include "gjp_ray.h"
#include "gjp_windows.h"

struct gjp_geometry {
  uint64_t id;                     // unique per handle (never reused)
  int n[3];
  double vs[3];
  double ctr[3];
  int n_views, n_u, n_v;
  int beam, weight;
  std::vector<double> views_world;  // as given
  std::vector<double> views_grid;   // n_views x 12, grid units
  std::vector<float> proj;          // n_views x 12: detector projection rows (u, v, w)
  gjp::GridGeom gg;
  // Every view has dv without in-plane component and no ray driven by axis 2:
  // the rays of a detector column share their in-plane coefficients, and the
  // adjoint uses the column-form gather.
  bool separable = false;
  // Rays per lane of the row forward (gjp_forward_rows.hip); 0: it cannot take the
  // geometry. rows_cost: its time per column and plane (rows_per_lane).
  int rows = 0;
  double rows_cost = 0.0;
  // General geometries: tile_v_log2 of the dealt tiles (FwdArgs::spread); deal: they are
  // the default (else groups of views with the set tile are).
  int deal_tile = 4;
  bool deal = false;
  bool free_gather = false;  // general geometry that adj_free_kernel takes
  // The adjoint runs as launch_adjoint_tiles, whose tiles of 64 and 128 voxels
  // along axis 2 need at most tile_rows[0] and tile_rows[1] detector rows.
  // axes: bit m set in a view's entry if axis m drives one of its columns.
  bool tiles = false;
  int tile_rows[2] = {0, 0};
  std::vector<uint8_t> axes;

  // device copies, per device (created on first use)
  struct Dev {
    double* views = nullptr;
    float* proj = nullptr;
  };
  static constexpr int kMaxDev = 64;
  mutable std::mutex mu;
  mutable Dev dev[kMaxDev];
};

namespace gjp {

// Status plumbing (defined in gjp_api.cpp).
int set_error(int status, const std::string& msg);

// Kernel timing registry (defined in gjp_api.cpp).
struct TimedLaunch {
  hipEvent_t start = nullptr, stop = nullptr;
  bool on = false;
};
TimedLaunch timing_begin(const char* name, hipStream_t s);
void timing_end(const char* name, TimedLaunch& t, hipStream_t s);

// Empty entries after each detector column in the column-form ray table
// (lets the adjoint read fixed-length candidate lists past a column's end).
constexpr int kColumnPad = 8;

// View splits of the tile adjoint. Both axes in one launch, and the views split
// so that it has about two rounds of workgroups (four per compute unit), with
// at least six views each (a split costs a partial volume's write and read):
// 64^3 / 64 views 193 us as two launches, 103, 62, 52, 48 and 57 us with 1, 2,
// 4, 8 and 16 splits; 128^3 / 12 views 76 us, then 58, 55 and 65 us with 1, 2
// and 4. Partial volumes of more than 128 MB, or one or two views: 0, a launch per
// driving axis into the volume itself (256^3 / 360 views 5.7 ms, 5.5 with one split;
// 512^3 80 ms; 256^3 / 2 views 83 us, 96 with one split; / 1 view at 45 degrees 74, 89).
inline int adjoint_tile_splits(const int* n, int n_views) {
  if (n_views <= 2) return 0;
  const size_t vol = (size_t)n[0] * n[1] * n[2] * sizeof(float);
  const size_t tiles = (size_t)((n[0] + kTileEdge - 1) / kTileEdge) *
                       ((n[1] + kTileEdge - 1) / kTileEdge) * ((n[2] + 127) / 128);
  size_t s = (2048 + 2 * tiles - 1) / (2 * tiles);
  const size_t by_views = n_views / 6 > 1 ? (size_t)n_views / 6 : 1;
  const size_t by_bytes = ((size_t)256 << 20) / (2 * vol);
  if (s > by_views) s = by_views;
  if (s > by_bytes) s = by_bytes;
  return (int)s;
}

// View splits of the gather of general geometries: about two rounds of workgroups
// (four per compute unit), at least six views each, partial volumes of at most
// 256 MiB.
inline int adjoint_free_splits(const int* n, int n_views) {
  const size_t vol = (size_t)n[0] * n[1] * n[2] * sizeof(float);
  const size_t tiles = (size_t)((n[0] + 15) / 16) * ((n[1] + 15) / 16) * ((n[2] + 7) / 8);
  size_t s = (2048 + tiles - 1) / tiles;
  const size_t by_views = n_views / 6 > 1 ? (size_t)n_views / 6 : 1;
  const size_t by_bytes = ((size_t)256 << 20) / vol;
  if (s > by_views) s = by_views;
  if (s > by_bytes) s = by_bytes;
  return s > 1 ? (int)s : 1;
}

// Launch configuration of the forward kernel.
struct FwdTile {
  int tile_v_log2 = 6;  // 6, 5, 4: 64, 32, 16 pixels along v per wavefront row;
                        // 7, 8: 128 / 192 pixels, two / three per lane (16-bit)
  int remap = 1;        // 1: contiguous tile ranges per XCD
  int view_group = 8;   // consecutive views that share each tile's turn
  int ru_group = 4;     // planes whose wide loads a lane issues together (2 or 4)
  int path = BY_RULE;   // kernels of the geometry's own (row forward, dealt tiles) or
                        // the padded copies in groups of views, with the tile above
  enum { BY_RULE, OWN, TILES };
};

// Arguments of one forward launch (one volume, a range of views).
struct FwdArgs {
  const void* vol_a;    // pair copy A (pairs along axis 1), padded element (0,0,0)
  const void* vol_b;    // pair copy B (pairs along axis 0), padded element (0,0,0)
  unsigned long long copy_bytes;  // bytes of one pair copy
  float* sino;          // sinogram of the whole geometry
  const double* views;  // device, n_views x 12 grid units
  GridGeom G;
  long long S0, S1;     // padded strides in pair elements
  int n_u, n_v;
  int tile_v_log2;
  int view_group;       // views interleaved per tile in the launch order
  int n_views;          // views of this launch
  int tiles_v, tiles_u, tiles_per_view;
  int remap;
  int ru_group;         // planes per load group of the row-uniform loop (2 or 4)
  // Row forward of column geometries (gjp_forward_rows.hip): rays per lane (0:
  // not used), tiles of 64 rows rays by four columns, and the caller's volume.
  int rows;
  const void* vol;
  // Launch order of general geometries (0: groups of views): view by view, units
  // of `spread` tiles (down a column of tiles, so that neighbours share lines in
  // L2) dealt to the eight XCDs in turn, starting one XCD later in every view.
  // tiles_per_view is rounded up to whole rounds.
  int spread;
};

// Device views of a geometry on the current device (uploads on first use).
int geometry_device(const gjp_geometry* g, const double** views, const float** proj);
// The same without uploading: GJP_EINVAL if there is no copy on this device.
int geometry_device_existing(const gjp_geometry* g, const double** views, const float** proj);

// Launchers (gjp_kernels.hip). Return a gjp_status.
int launch_pad(const void* src, void* copy_a, void* copy_b, int dtype, const int n[3],
               hipStream_t s);
int launch_zero_ints(int* p, int n, hipStream_t s);
int launch_sart_residual(long long n, const float* b, const float* ax, const float* w,
                         float* out, hipStream_t s);
int launch_sart_update(long long n, float* x, const float* bp, const float* c, float lam,
                       int nonneg, hipStream_t s);
int launch_forward(const FwdArgs& a, int dtype, int weight, bool idx64, int n_views,
                   hipStream_t s);
// Row forward (gjp_forward_rows.hip; a.rows rays per lane), launched within
// launch_forward and launch_batched_forward.
void launch_forward_rows(const FwdArgs& a, int dtype, int weight, unsigned grid, hipStream_t s);
int launch_forward_naive(const GridGeom& G, const double* views, const void* vol, int dtype,
                         int weight, int n_views, int n_u, int n_v, float* sino, hipStream_t s);
int launch_adjoint_table(const gjp_geometry* g, const double* views, const float* sino,
                         int view0, int n_chunk, float4* table, float4* cols, int* mask,
                         hipStream_t s);
// Column map of the value-table adjoint: every ray v of detector column u
// has driving axis m, in-plane coordinate fma(i, ga, ca) on plane i and
// axis-2 coordinate A + v B there, with t = (i - sm) inv_rm, A = a0 + t a1,
// B = b0 + t b1.
struct ResCol {
  int m;  // driving axis (0 or 1); -1: no samples
  float ca, ga, pad;
  double sm, inv_rm;
  double a0, a1, b0, b1;
};
int launch_adjoint_value_table(const gjp_geometry* g, const double* views, const float* sino,
                               int view0, int n_chunk, float* vals, ResCol* cols, int* mask,
                               hipStream_t s);
// Tile adjoint of column geometries (gjp_adjoint_tiles.hip): n_views views
// (views, proj: the first one's entries) of rays scaled by their step lengths
// (launch_adjoint_scale), driven by axis 0 (axes: bit 0), 1 (bit 1) or both; adds to vol
// or overwrites it. part: scratch for 2 x splits partial volumes, splits =
// adjoint_tile_splits; null for 0 splits.
int launch_adjoint_scale(const gjp_geometry* g, const double* views, const float* sino, int n_views,
                         float* out, hipStream_t s);
int launch_adjoint_tiles(const gjp_geometry* g, const double* views, const float* proj,
                         const float* rays, int n_views, int axes, bool accumulate, float* vol,
                         float* part, int splits, hipStream_t s);
// Sum of partial volumes (slice floats each), added to vol if accumulate.
int launch_adjoint_sum(const float* part, size_t slice, int n_slices, bool accumulate, float* vol,
                       hipStream_t s);
// Gather of general geometries (g->free_gather, gjp_adjoint_free.hip) from
// adj_table_kernel's rays and axes of n_views views; proj: the first one's. part:
// splits partial volumes, splits = adjoint_free_splits, used above 1.
int launch_adjoint_free(const gjp_geometry* g, const float* proj, const float4* table,
                        const int* mask, int n_views, bool accumulate, float* vol, float* part,
                        int splits, hipStream_t s);
// launch_adjoint_value_table without cols writes launch_adjoint_scale's rays.
// launch_adjoint_gather, by the pointers that are not null:
//   vals, rcols     column gather from the value table
//   vals            tile adjoint; vals: the scaled rays, cols: scratch for the partial
//                   volumes of adjoint_tile_splits, or null (none, also if those are 0)
//   table           column geometries: column gather from the ray table (and cols);
//                   general ones: cube gather (cols: scratch for the partial volumes of
//                   adjoint_free_splits, or null: none) or tile splat
int launch_adjoint_gather(const gjp_geometry* g, const float* proj, const float4* table,
                          const float4* cols, const float* vals, const ResCol* rcols,
                          const int* mask, int view0, int c0, int n_chunk, bool accumulate,
                          float* vol, hipStream_t s);

// Batched forward (gjp_batched.cpp / gjp_kernels.hip).
struct BatchInst {
  FwdArgs a;
  const void* src;      // caller volume (unpadded)
  void* padded;         // plan-owned pair copies A and B (A at the start)
  int n_views;
  int dtype, weight, idx64;
  long long padded_elems;
};
int launch_batched_pad(const BatchInst* d_insts, int n_inst, hipStream_t s);
// Instance class of the batched launch: storage type, weight, 64-bit
// addressing and three rays per lane (192-wide tiles) or one.
inline int batch_class(int dtype, int weight, int idx64, int triple) {
  return ((dtype * 2 + weight) * 2 + idx64) * 2 + triple;
}
// ... and of the instances that the row forward takes.
inline int batch_rows_class(int dtype, int weight) { return 24 + dtype * 2 + weight; }
constexpr int kBatchClasses = 30;
// Queues per class of the batched launch: one per XCD.
constexpr int kBatchQueues = 8;
// One class's persistent launch: items of its kBatchQueues queues, queue q =
// d_items[d_qoff[q] .. d_qoff[q + 1]), counters d_counters[0 .. kBatchQueues).
int launch_batched_forward(const BatchInst* d_insts, const uint2* d_items, const int* d_qoff,
                           int* d_counters, int grid, int cls, hipStream_t s);
int batched_grid_size(int cls);
void launch_batched_rows(const BatchInst* d_insts, const uint2* d_items, const int* d_qoff,
                         int* d_counters, int grid, int dtype, int weight, hipStream_t s);
const void* batched_rows_function(int dtype, int weight);  // its kernel

size_t dtype_size(int dtype);

// Detector pixels along v per wavefront row of a forward tile code, and
// detector columns per workgroup tile.
inline int tile_v_pixels(int tile_v_log2) { return tile_v_log2 == 8 ? 192 : 1 << tile_v_log2; }
inline int tile_u_columns(int tile_v_log2) { return tile_v_log2 >= 7 ? 4 : 256 >> tile_v_log2; }

// Fixed device scratch of gjp_forward_project_noalloc (gjp_kernels.hip): its
// size, and its address on the current device (looked up once per device).
constexpr size_t kNoAllocScratchBytes = (size_t)64 << 20;
int noalloc_scratch(void** ptr);

}  // namespace gjp

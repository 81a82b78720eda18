// Driver of the library's host rules (built by tests/test_host_planning_cpu.py from
// csrc/gjp_api.cpp for the host only): which kernel a geometry is sent to, and whether
// what that kernel copies to LDS fits for every geometry that is sent to it. The
// kernels' launchers are stand-ins.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <vector>

#include "gjp.h"
#include "gjp_internal.h"
#include "gjp_windows.h"

namespace gjp {
int launch_pad(const void*, void*, void*, int, const int*, hipStream_t) { return 0; }
int launch_zero_ints(int*, int, hipStream_t) { return 0; }
int launch_sart_residual(long long, const float*, const float*, const float*, float*,
                         hipStream_t) { return 0; }
int launch_sart_update(long long, float*, const float*, const float*, float, int, hipStream_t) {
  return 0;
}
static int g_forward_rows = -1;
int launch_forward(const FwdArgs& a, int, int, bool, int, hipStream_t) {
  g_forward_rows = a.rows;
  return 0;
}
int launch_forward_naive(const GridGeom&, const double*, const void*, int, int, int, int, int,
                         float*, hipStream_t) { return 0; }
int launch_adjoint_table(const gjp_geometry*, const double*, const float*, int, int, float4*,
                         float4*, int*, hipStream_t) { return 0; }
struct Gather {
  const void *table, *cols, *vals, *rcols;
  int view0, c0, n;
  bool accumulate;
};
static std::vector<Gather> g_gathers;
int launch_adjoint_gather(const gjp_geometry*, const float*, const float4* table,
                          const float4* cols, const float* vals, const ResCol* rcols, const int*,
                          int view0, int c0, int n, bool accumulate, float*, hipStream_t) {
  g_gathers.push_back({table, cols, vals, rcols, view0, c0, n, accumulate});
  return 0;
}
int launch_adjoint_value_table(const gjp_geometry*, const double*, const float*, int, int, float*,
                               ResCol*, int*, hipStream_t) { return 0; }
int launch_batched_pad(const BatchInst*, int, hipStream_t) { return 0; }
int launch_batched_forward(const BatchInst*, const uint2*, const int*, int*, int, int,
                           hipStream_t) { return 0; }
int batched_grid_size(int) { return 1; }
size_t dtype_size(int dtype) { return dtype == 0 ? 4 : 2; }
int noalloc_scratch(void**) { return -1; }
}  // namespace gjp

// Device memory, as far as the host path takes it: blocks of a given total at most, not
// backed by memory of their size (the stand-ins read none).
static size_t g_free_bytes = (size_t)1 << 60, g_largest = 0;
static std::map<void*, size_t> g_blocks;
static hipError_t take(void** p, size_t n) {
  if (n > g_free_bytes) return hipErrorOutOfMemory;
  g_free_bytes -= n;
  g_largest = std::max(g_largest, n);
  *p = aligned_alloc(256, 256);
  g_blocks[*p] = n;
  return hipSuccess;
}
static hipError_t give(void* p) {
  if (!p) return hipSuccess;
  g_free_bytes += g_blocks.at(p);
  g_blocks.erase(p);
  free(p);
  return hipSuccess;
}
extern "C" {
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return take(p, n); }
hipError_t hipFree(void* p) { return give(p); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return take(p, n); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return give(p); }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t*, int) { return hipErrorNotSupported; }
}

static int bad = 0;
#define CHECK(c)                                                   \
  do {                                                             \
    if (!(c)) {                                                    \
      if (bad < 20) fprintf(stderr, "line %d: %s\n", __LINE__, #c); \
      ++bad;                                                       \
    }                                                              \
  } while (0)

static uint64_t g_state = 88172645463325252ull;
static double uniform(double a, double b) {
  g_state ^= g_state << 13;
  g_state ^= g_state >> 7;
  g_state ^= g_state << 17;
  return a + (b - a) * ((double)(g_state >> 11) / 9007199254740992.0);
}
static double loguniform(double a, double b) { return exp(uniform(log(a), log(b))); }
static int integer(double a, double b) { return (int)floor(loguniform(a, b + 0.999)); }

static gjp_geometry* make(const int* n, int beam, int n_views, int n_u, int n_v,
                          const double* views) {
  gjp_geometry_desc d;
  memset(&d, 0, sizeof(d));
  for (int k = 0; k < 3; ++k) {
    d.vol_shape[k] = n[k];
    d.voxel_size[k] = 1.0;
  }
  d.n_views = n_views;
  d.n_u = n_u;
  d.n_v = n_v;
  d.beam = beam;
  d.views = views;
  gjp_geometry* g = nullptr;
  return gjp_create_geometry(&d, &g) == GJP_OK ? g : nullptr;
}

// A column geometry's view: source `dist` from the centre at angle th and height zs (cone;
// parallel: climb zs per unit), detector `len` away, pitches pu and pv, rows shifted by
// `v_off` pixels, columns climbing su along axis 2.
static void column_view(int beam, double th, double dist, double zs, double len, double pu,
                        double pv, double su, int n_u, int n_v, double v_off, double* o) {
  const double c = cos(th), s = sin(th);
  const double du[3] = {-pu * s, pu * c, su}, dv[3] = {0.0, 0.0, pv};
  const double first[3] = {beam == GJP_CONE ? dist * c : -c, beam == GJP_CONE ? dist * s : -s, zs};
  const double mid[3] = {(dist - len) * c, (dist - len) * s, v_off * pv};
  for (int k = 0; k < 3; ++k) {
    o[k] = first[k];
    o[3 + k] = (beam == GJP_CONE ? mid[k] : 0.0) - 0.5 * (n_u - 1) * du[k] -
               0.5 * (n_v - 1) * dv[k] + (k == 2 && beam != GJP_CONE ? mid[2] : 0.0);
    o[6 + k] = du[k];
    o[9 + k] = dv[k];
  }
}

// Every window of the row forward lies in its LDS row, on every plane that the sampling
// loop takes.
static void check_row_windows(const gjp_geometry& g) {
  const int R = g.rows;
  for (int view = 0; view < g.n_views; ++view) {
    const double* v = g.views_grid.data() + 12 * (size_t)view;
    const bool cone = g.beam == GJP_CONE;
    for (int u = 0; u < g.n_u; ++u) {
      const double d0 = v[3] + u * v[6], d1 = v[4] + u * v[7], d2 = v[5] + u * v[8];
      const double s0 = cone ? v[0] : d0, s1 = cone ? v[1] : d1;
      const double r0 = cone ? d0 - v[0] : v[0], r1 = cone ? d1 - v[1] : v[1];
      const bool m1 = fabs(r1) > fabs(r0);
      const double sm = m1 ? s1 : s0, rm = m1 ? r1 : r0;
      const int nm = m1 ? g.n[1] : g.n[0];
      if (rm == 0.0) continue;
      for (int v0 = 0; v0 < g.n_v; v0 += 64 * R) {
        const int last = std::min(g.n_v - v0, 64 * R) - 1;
        const double irm = 1.0 / rm;
        const double A = cone ? v[2] : d2 + v0 * v[11], B = cone ? 0.0 : v[11];
        const double C = (cone ? d2 + v0 * v[11] - v[2] : v[2]) * irm, D = cone ? v[11] * irm : 0.0;
        // blocks may begin at any plane and hold up to kRowPlanes of the grid's
        for (int p0 = 0; p0 < nm; p0 += std::max(1, nm / 7)) {
          const int np = std::min(gjp::kRowPlanes, nm - p0);
          const double t0 = p0 - sm;
          gjp::RowWindow w;
          if (!gjp::row_window(A, B, C, D, t0, gjp::row_planes(np), last, g.n[2], w)) continue;
          CHECK(w.pad % 4 == 0 && w.zd >= 0 && w.need >= 1);
          CHECK(w.zd + w.need <= g.n[2]);
          CHECK(w.pad + ((w.need + 3) & ~3) <= gjp::kRowEntries);
          for (int i = 0; i < gjp::row_planes(np); ++i)
            for (int k = 0; k <= last; k += std::max(1, last)) {
              const double e = floor(A + k * B + (t0 + i) * (C + k * D)) - w.zd + w.pad;
              CHECK(e >= 0 && e + 1 < gjp::kRowEntries);
            }
        }
      }
    }
  }
}

static int rows_main() {
  int taken = 0, wide = 0;
  for (int trial = 0; trial < 4000; ++trial) {
    const int n[3] = {integer(1, 40), integer(1, 40), integer(2, 300)};
    const int beam = trial % 3 == 0 ? GJP_PARALLEL : GJP_CONE, n_v = integer(2, 600), n_u = 5;
    const double reach = 0.5 * std::max(n[0], n[1]);
    const double dist = reach + loguniform(2.0, 400.0), len = dist * uniform(1.05, 3.0);
    const double climb = uniform(-0.99, 0.99);
    double views[24];
    for (int k = 0; k < 2; ++k)
      column_view(beam, uniform(0.0, 6.28), dist,
                  beam == GJP_CONE ? climb * dist * uniform(0.0, 1.0) : climb * 0.7, len,
                  loguniform(0.2, 3.0), loguniform(0.05, 6.0) * (trial & 1 ? 1 : -1), 0.0, n_u, n_v,
                  uniform(-0.5, 0.5) * n_v, views + 12 * k);
    gjp_geometry* g = make(n, beam, 2, n_u, n_v, views);
    CHECK(g != nullptr);
    if (g->rows) {
      ++taken;
      check_row_windows(*g);
    }
    gjp_destroy_geometry(g);
  }
  // a thin volume seen steeply from below: windows that the planes past the grid widen
  {
    const int n[3] = {4, 4, 240};
    double v[12];
    for (double pv = 3.0; pv < 3.8; pv += 0.002) {
      for (double z = -240.0; z < 0.0; z += 8.0) {
        column_view(GJP_CONE, M_PI, 238.0, z, 476.0, 1.0, pv, 0.0, 1, 256, 0.0, v);
        gjp_geometry* g = make(n, GJP_CONE, 1, 1, 256, v);
        if (g->rows) {
          ++wide;
          check_row_windows(*g);
        }
        gjp_destroy_geometry(g);
      }
    }
  }
  CHECK(taken > 400 && wide > 1000);
  return 0;
}

// Every window of the tile adjoint fits, and holds every ray that has weight in its tile.
static void check_tile_windows(const gjp_geometry& g, long long* windows) {
  const bool cone = g.beam == GJP_CONE;
  const bool one = g.n[2] <= 64 || g.tile_rows[1] > gjp::kTileMaxRows;
  const int zt = one ? 64 : 128, E = gjp::kTileEdge;
  for (int view = 0; view < g.n_views; ++view) {
    const double* v = g.views_grid.data() + 12 * (size_t)view;
    const float* Q = g.proj.data() + 12 * (size_t)view;
    const bool flip = v[11] < 0.0;
    for (int m = 0; m < 2; ++m)
      for (int p0 = 0; p0 < g.n[m]; p0 += E)
        for (int ra0 = 0; ra0 < g.n[1 - m]; ra0 += E)
          for (int z0 = 0; z0 < g.n[2]; z0 += zt) {
            const gjp::TileWindow w =
                gjp::tile_window(v, Q, cone, g.n_u, g.n_v, m, p0, ra0, z0, zt);
            const bool used = w.uhi >= w.ulo && w.any && w.v0 < g.n_v && w.v0 + w.rows > 0;
            if (used) {
              ++*windows;
              CHECK(w.rows <= gjp::kTileMaxRows);
            }
            for (int u = 0; u < g.n_u; u += 1 + g.n_u / 40) {
              const gjp::Column c = gjp::column_line(v, cone, u);
              if (c.m != m) continue;
              const double sm = m == 0 ? c.s0 : c.s1, sa = m == 0 ? c.s1 : c.s0;
              const double rm = m == 0 ? c.r0 : c.r1, ra = m == 0 ? c.r1 : c.r0;
              for (int i = p0; i < std::min(p0 + E, g.n[m]); ++i) {
                const double pa = sa + (i - sm) * (ra / rm), t = (i - sm) / rm;
                if (!(pa > ra0 - 1.0 && pa < ra0 + E)) continue;
                // rays of the column within a voxel of the tile along axis 2
                const double d2 = v[5] + u * v[8];
                const double A = cone ? v[2] + t * (d2 - v[2]) : d2 + t * v[2];
                const double B = cone ? t * v[11] : v[11];
                double k0 = (z0 - 1.0 - A) / B, k1 = (z0 + zt - A) / B;
                if (k0 > k1) std::swap(k0, k1);
                k0 = std::max(ceil(k0), 0.0);
                k1 = std::min(floor(k1), g.n_v - 1.0);
                if (k0 > k1) continue;
                CHECK(used && u >= w.ulo && u <= w.uhi);
                if (flip) {
                  const double h = k0;
                  k0 = g.n_v - 1 - k1;
                  k1 = g.n_v - 1 - h;
                }
                CHECK(k0 >= w.v0 && k1 < w.v0 + w.rows);
              }
            }
          }
  }
}

static int tiles_main() {
  int taken = 0, refused = 0;
  long long windows = 0;
  for (int trial = 0; trial < 3000; ++trial) {
    const int n[3] = {integer(1, 40), integer(1, 40), integer(2, 300)};
    const int beam = trial % 3 == 0 ? GJP_PARALLEL : GJP_CONE;
    const int n_v = integer(2, 60), n_u = integer(1, 200);
    const double reach = 0.5 * std::max(n[0], n[1]);
    const double dist = reach + loguniform(4.0, 400.0), len = dist * uniform(1.05, 3.0);
    const double pu = loguniform(0.05, 3.0), climb = uniform(-0.99, 0.99);
    // columns that climb: along the detector, or more than it advances
    const double su = trial % 4 == 0 ? pu * loguniform(0.1, 30.0) * (trial & 8 ? 1 : -1) : 0.0;
    double views[24];
    for (int k = 0; k < 2; ++k)
      column_view(beam, uniform(0.0, 6.28), dist,
                  beam == GJP_CONE ? climb * dist * uniform(0.0, 1.0) : climb * 0.7, len, pu,
                  loguniform(0.01, 6.0) * (trial & 1 ? 1 : -1), su, n_u, n_v,
                  uniform(-0.5, 0.5) * n_v, views + 12 * k);
    if (trial % 5 == 0) {  // detectors nearly along the rays
      const double a = uniform(1.4, 1.56);
      for (int k = 0; k < 2; ++k) {
        double* o = views + 12 * k;
        const double x = cos(a) * o[6] - sin(a) * o[7], y = sin(a) * o[6] + cos(a) * o[7];
        for (int j = 0; j < 2; ++j) o[3 + j] -= 0.5 * (n_u - 1) * ((j ? y : x) - o[6 + j]);
        o[6] = x;
        o[7] = y;
      }
    }
    gjp_geometry* g = make(n, beam, 2, n_u, n_v, views);
    CHECK(g != nullptr);
    if (g->tiles) {
      ++taken;
      check_tile_windows(*g, &windows);
    } else if (g->separable) {
      ++refused;
    }
    gjp_destroy_geometry(g);
  }
  // columns ten voxels apart along axis 2, rays a fiftieth: more rows than fit
  {
    const int n[3] = {24, 24, 60};
    double v[12];
    for (double su = 0.0; su <= 12.0; su += 0.5) {
      column_view(GJP_PARALLEL, 0.3, 0.0, 0.0, 0.0, 1.0, 0.02, su, 40, 3000, 0.0, v);
      gjp_geometry* g = make(n, GJP_PARALLEL, 1, 40, 3000, v);
      CHECK(su > 0.0 || g->tiles);
      if (g->tiles) check_tile_windows(*g, &windows);
      gjp_destroy_geometry(g);
    }
  }
  CHECK(taken > 500 && windows > 4000 && refused > 20);
  return 0;
}

// One call of the adjoint with `room` bytes free: its status, the launches it made, and
// that it gave back what it took.
static gjp_status back(const gjp_geometry* g, size_t room) {
  gjp::g_gathers.clear();
  g_largest = 0;
  const double* views;
  const float* proj;
  g_free_bytes = (size_t)1 << 60;
  CHECK(gjp::geometry_device(g, &views, &proj) == GJP_OK);
  g_free_bytes = room;
  const gjp_status st = gjp_back_project(g, (const float*)16, (float*)16, nullptr);
  CHECK(g_free_bytes == room);
  g_free_bytes = (size_t)1 << 60;
  if (st != GJP_OK) return st;
  // every view once, in order; all but the first launch add
  int next = 0;
  for (const auto& q : gjp::g_gathers) {
    CHECK(q.view0 + q.c0 == next && q.accumulate == (next > 0));
    next += q.n;
  }
  CHECK(next == g->n_views);
  return st;
}

static int scratch_main() {
  const int n[3] = {64, 64, 64};
  std::vector<double> v(12 * 40);
  {  // scaled rays of a view 64 MiB: 32 views in 2 GiB, then 8; two partial volumes per split
    CHECK(gjp_views_circular_cone(40, 256, 512, 0.05, 0.15, 4096, 4096, v.data()) == GJP_OK);
    gjp_geometry* g = make(n, GJP_CONE, 40, 4096, 4096, v.data());
    CHECK(g && g->tiles);
    const size_t view = (size_t)4096 * 4096 * 4, vol = (size_t)64 * 64 * 64 * 4;
    CHECK(back(g, (size_t)1 << 40) == GJP_OK && gjp::g_gathers.size() == 2);
    CHECK(gjp::g_gathers[0].n == 32 && gjp::g_gathers[0].cols && !gjp::g_gathers[0].rcols);
    CHECK(g_largest >= 32 * view + 2 * gjp::adjoint_tile_splits(n, 32) * vol);
    // less room: quarters of the views (one or two have no partial volumes)
    CHECK(back(g, 20 * view) == GJP_OK && gjp::g_gathers[0].n == 8 && gjp::g_gathers[0].cols);
    CHECK(back(g, 3 * view) == GJP_OK && gjp::g_gathers[0].n == 2 && !gjp::g_gathers[0].cols);
    CHECK(back(g, view) == GJP_OK && gjp::g_gathers.size() == 40 && !gjp::g_gathers[0].cols);
    CHECK(back(g, view - 1) == GJP_ENOMEM);
    gjp_destroy_geometry(g);
  }
  {  // fan beams, one row: no more columns per launch than 2^32 threads scale
    const int flat[3] = {64, 64, 1};
    std::vector<double> w(12 * 20000);
    CHECK(gjp_views_circular_cone(20000, 256, 512, 0.03, 1.0, 4096, 1, w.data()) == GJP_OK);
    gjp_geometry* g = make(flat, GJP_CONE, 20000, 4096, 1, w.data());
    CHECK(g && g->tiles);
    CHECK(back(g, (size_t)1 << 40) == GJP_OK && gjp::g_gathers.size() > 1);
    for (const auto& q : gjp::g_gathers) CHECK(((long long)q.n * 4096 + 3) / 4 * 256 < (1ll << 32));
    gjp_destroy_geometry(g);
  }
  {  // general geometries: what sufficed for the ray table suffices
    const int big[3] = {128, 128, 128};
    CHECK(gjp_views_circular_cone(40, 512, 1024, 2, 2, 200, 200, v.data()) == GJP_OK);
    for (int k = 0; k < 40; ++k) v[12 * k + 9] = 0.3;
    gjp_geometry* g = make(big, GJP_CONE, 40, 200, 200, v.data());
    CHECK(g && g->free_gather);
    const size_t table = (size_t)40 * 200 * 200 * 32, vol = (size_t)128 * 128 * 128 * 4;
    const size_t splits = gjp::adjoint_free_splits(big, 40);
    CHECK(splits > 1);
    CHECK(back(g, (size_t)1 << 40) == GJP_OK && gjp::g_gathers[0].cols);
    CHECK(g_largest == table + splits * vol);
    CHECK(back(g, table + splits * vol + 4096) == GJP_OK && gjp::g_gathers[0].cols);
    CHECK(back(g, table + splits * vol - 1) == GJP_OK && !gjp::g_gathers[0].cols);
    CHECK(back(g, table + 4096) == GJP_OK && !gjp::g_gathers[0].cols);
    CHECK(back(g, table - 1) == GJP_ENOMEM);
    gjp_destroy_geometry(g);
  }
  return 0;
}

// What the geometry's creation found from a few columns of each view against all of them.
static int columns_main() {
  int yes = 0, no = 0, tiles = 0;
  for (int trial = 0; trial < 20000; ++trial) {
    const int n[3] = {integer(4, 40), integer(4, 40), integer(4, 100)};
    const int n_u = integer(40, 400), n_v = integer(2, 200);
    const double dist = loguniform(6.0, 200.0), len = dist * uniform(1.02, 2.0);
    double views[12];
    column_view(GJP_CONE, uniform(0.0, 6.28), dist, uniform(-0.5, 0.5) * dist, len,
                loguniform(0.02, 4.0), loguniform(0.02, 4.0) * (trial & 1 ? 1 : -1),
                trial % 3 ? 0.0 : uniform(-0.5, 0.5), n_u, n_v, uniform(-0.5, 0.5) * n_v, views);
    if (trial % 4 == 0) {  // detectors of any direction in the plane
      const double a = uniform(-1.57, 1.57), x = cos(a) * views[6] - sin(a) * views[7],
                   y = sin(a) * views[6] + cos(a) * views[7];
      for (int j = 0; j < 2; ++j) views[3 + j] -= 0.5 * (n_u - 1) * ((j ? y : x) - views[6 + j]);
      views[6] = x;
      views[7] = y;
    }
    gjp_geometry* g = make(n, GJP_CONE, 1, n_u, n_v, views);
    CHECK(g != nullptr);
    const double* o = g->views_grid.data();
    bool separable = o[9] == 0.0 && o[10] == 0.0;
    bool used[2] = {false, false}, front = true;
    for (int iu = 0; iu < n_u; ++iu) {
      const double r[2] = {o[3] + iu * o[6] - o[0], o[4] + iu * o[7] - o[1]};
      const double M = fmax(fabs(r[0]), fabs(r[1]));
      const double z0 = o[5] + iu * o[8] - o[2], z1 = o[5] + iu * o[8] + (n_v - 1) * o[11] - o[2];
      if (!(fmax(fabs(z0), fabs(z1)) * (1.0 + 1e-9) < M)) separable = false;
      const int m = fabs(r[1]) > fabs(r[0]) ? 1 : 0;
      used[m] = true;
      if (!((o[m] < -3.0 && r[m] > 0.0) || (o[m] > n[m] + 20.0 && r[m] < 0.0))) front = false;
    }
    CHECK(g->separable == separable);
    if (g->tiles) {
      ++tiles;
      CHECK(front);
    }
    ++(separable ? yes : no);
    gjp_destroy_geometry(g);
  }
  CHECK(yes > 2000 && no > 2000 && tiles > 500);
  return 0;
}

// Whether a forward runs without padded copies (set tile shape; 0: the default).
static bool rows_taken(const gjp_geometry* g, int dtype, int tile) {
  CHECK(gjp_set_forward_tile(g, dtype, tile, 8, 4) == GJP_OK);
  g_largest = 0;
  gjp::g_forward_rows = -1;
  CHECK(gjp_forward_project(g, (const void*)16, dtype, (float*)16, nullptr) == GJP_OK);
  CHECK(gjp_set_forward_tile(g, dtype, 0, 8, 4) == GJP_OK);
  return gjp::g_forward_rows > 0;
}

// The kernels that geometries of each kind are sent to.
static int dispatch_main() {
  const int n[3] = {64, 60, 70};
  std::vector<double> v(12 * 30);
  gjp_geometry* g;
  CHECK(gjp_views_circular_cone(30, 256, 512, 2, 2, 64, 64, v.data()) == GJP_OK);
  g = make(n, GJP_CONE, 30, 64, 64, v.data());  // ordinary circular scan
  CHECK(g && g->separable && g->rows > 0 && g->tiles && !g->free_gather);
  CHECK(rows_taken(g, GJP_F32, 0) && rows_taken(g, GJP_BF16, 0));
  gjp_destroy_geometry(g);
  {  // columns of 128 rays: rows for FP32, small 16-bit copies for 16 bits; 64: copies
    const int m[3] = {128, 128, 128};
    std::vector<double> w(12 * 200);
    for (int n_v : {64, 128, 192}) {
      CHECK(gjp_views_circular_cone(200, 512, 768, 1.0, 1.55 * 128 / n_v, 192, n_v, w.data()) ==
            GJP_OK);
      g = make(m, GJP_CONE, 200, 192, n_v, w.data());
      CHECK(g && g->rows > 0 && rows_taken(g, GJP_F32, 0) == (n_v > 64));
      CHECK(rows_taken(g, GJP_F16, 0) == (n_v > 128));
      // a set tile of 192 rays, of which the copies' kernel would leave most idle
      CHECK(n_v == 64 || (rows_taken(g, GJP_F32, 192) && rows_taken(g, GJP_BF16, 192)));
      gjp_destroy_geometry(g);
    }
  }
  {  // half-filled wavefronts of rows: only where the call is over before the host is
    const int m[3] = {45, 58, 50};
    std::vector<double> w(12 * 123);
    for (int n_views : {40, 123}) {
      CHECK(gjp_views_circular_cone(n_views, 180, 270, 1.3, 2.0, 71, 40, w.data()) == GJP_OK);
      g = make(m, GJP_CONE, n_views, 71, 40, w.data());
      for (int dtype : {GJP_F32, GJP_BF16, GJP_F16})
        CHECK(g && g->rows > 0 && rows_taken(g, dtype, 0) == (n_views == 40));
      gjp_destroy_geometry(g);
    }
  }
  CHECK(gjp_views_parallel(30, 1, 1, 90, 80, v.data()) == GJP_OK);
  g = make(n, GJP_PARALLEL, 30, 90, 80, v.data());
  CHECK(g && g->separable && g->rows > 0 && g->tiles && !g->free_gather);
  gjp_destroy_geometry(g);
  CHECK(gjp_views_circular_cone(30, 48, 512, 2, 0.1, 64, 64, v.data()) == GJP_OK);
  g = make(n, GJP_CONE, 30, 64, 64, v.data());  // sources too near for the tiles
  CHECK(g && g->separable && !g->tiles && !g->free_gather);
  gjp_destroy_geometry(g);
  CHECK(gjp_views_circular_cone(30, 256, 512, 2, 2, 64, 64, v.data()) == GJP_OK);
  for (int k = 0; k < 30; ++k) v[12 * k + 9] = 0.3;  // tilted detectors
  g = make(n, GJP_CONE, 30, 64, 64, v.data());
  CHECK(g && !g->separable && !g->rows && !g->tiles && g->free_gather);
  gjp_destroy_geometry(g);
  CHECK(gjp_views_circular_cone(30, 44, 80, 2, 1.5, 64, 90, v.data()) == GJP_OK);
  g = make(n, GJP_CONE, 30, 64, 90, v.data());  // columns along axis 2, some rays driven by it
  CHECK(g && !g->separable && !g->deal);
  gjp_destroy_geometry(g);
  CHECK(gjp_views_circular_cone(30, 256, 512, 2, 2, 64, 64, v.data()) == GJP_OK);
  for (int k = 0; k < 30; ++k) v[12 * k + 9] = 0.3;
  {  // many views of many tiles, up to what one launch takes
    std::vector<double> w(12 * 1500);
    CHECK(gjp_views_circular_cone(1500, 256, 512, 0.2, 0.2, 1500, 1500, w.data()) == GJP_OK);
    for (int k = 0; k < 1500; ++k) w[12 * k + 9] = 0.03;
    g = make(n, GJP_CONE, 1500, 1500, 1500, w.data());
    CHECK(g && !g->separable && g->deal);
    gjp_destroy_geometry(g);
    g = make(n, GJP_CONE, 1500, 1800, 1800, w.data());
    CHECK(g && !g->separable && !g->deal);
    gjp_destroy_geometry(g);
  }
  const int det[][4] = {{64, 64, 0, 4}, {180, 180, 1, 4}, {1, 200, 1, 6}, {7, 100, 1, 5},
                        {200, 3, 1, 4}, {30, 30, 1, 4}, {40, 300, 1, 4}};
  for (const auto& d : det) {
    g = make(n, GJP_CONE, 30, d[0], d[1], v.data());
    CHECK(g && g->deal == (d[2] != 0) && g->deal_tile == d[3]);
    gjp_destroy_geometry(g);
  }
  for (int k = 0; k < 30; ++k)  // and sources inside the grid
    for (int j = 0; j < 3; ++j) v[12 * k + j] *= 0.05;
  g = make(n, GJP_CONE, 30, 64, 64, v.data());
  CHECK(g && !g->separable && !g->rows && !g->tiles && !g->free_gather);
  gjp_destroy_geometry(g);
  return 0;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "rows")) rows_main();
  else if (!strcmp(what, "tiles")) tiles_main();
  else if (!strcmp(what, "scratch")) scratch_main();
  else if (!strcmp(what, "dispatch")) dispatch_main();
  else if (!strcmp(what, "columns")) columns_main();
  else {
    fprintf(stderr, "unknown part %s\n", what);
    return 2;
  }
  printf(bad ? "planning driver %s: FAILED (%d)\n" : "planning driver %s: ok\n", what, bad);
  return bad != 0;
}

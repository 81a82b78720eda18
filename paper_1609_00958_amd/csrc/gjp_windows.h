// gjp_windows.h -- windows of voxels and of detector rows that the kernels of column
// geometries copy to LDS, shared by the kernels and by the host, whose rules send a
// geometry to a kernel only where every window fits.
#pragma once

#include <math.h>

#include "gjp_ray.h"

namespace gjp {

// Row forward (gjp_forward_rows.hip). Planes that share a window of voxels along axis 2
// (16: 2% slower at 512^3; a longer block widens the windows of steep rays), entries of
// a combined row in LDS, and the multiple of planes that the sampling loop takes.
constexpr int kRowPlanes = 32;
constexpr int kRowEntries = 512;
constexpr int kRowStep = 4;

// Voxels along axis 2 that rays 0 .. last of a wavefront span on `planes` planes from
// the one at t0 on: ray k lies at (A + k B) + t (C + k D). Entries pad, pad + 1, ... of
// the LDS row hold voxels zd .. zd + need - 1; entry 0 is voxel zd - pad.
struct RowWindow {
  int zd, need, pad;
  bool border;  // rays reach beside the grid
};

// False if no ray comes within a voxel of the grid. Coordinates are linear in the ray
// and in the plane, so the corners bound them. Voxels are loaded from one on that
// leaves a multiple of four to the row's end (or is its first).
GJP_HD bool row_window(double A, double B, double C, double D, double t0, int planes, int last,
                       int n2, RowWindow& w) {
  const double t1 = t0 + (double)(planes - 1), kl = (double)last;
  const double c00 = A + t0 * C, c01 = A + t1 * C;
  const double c10 = c00 + kl * (B + t0 * D), c11 = c01 + kl * (B + t1 * D);
  const double zmin = fmin(fmin(c00, c01), fmin(c10, c11));
  const double zmax = fmax(fmax(c00, c01), fmax(c10, c11));
  if (!(zmax > -1.0 && zmin < (double)n2)) return false;
  const int lo = (int)floor(zmin - 0.01), hi = (int)floor(zmax + 0.01) + 1;
  const int first = lo > 0 ? lo : 0;
  const int zd = first - ((first - n2) & 3);
  w.zd = zd > 0 ? zd : 0;
  w.need = (hi < n2 - 1 ? hi : n2 - 1) - w.zd + 1;
  w.pad = (w.zd - lo > 0 ? w.zd - lo + 3 : 3) & ~3;
  w.border = lo < 0 || hi >= n2;
  return true;
}

// Planes whose windows a block of np planes needs: the loop's, in whole steps.
GJP_HD int row_planes(int np) { return (np + kRowStep - 1) & ~(kRowStep - 1); }

// Tile adjoint (gjp_adjoint_tiles.hip): voxels of a tile along axes 0 and 1, the
// detector rows of one column that it can stage, and the detector columns that one
// launch scales (a wavefront each, below 2^32 threads).
constexpr int kTileEdge = 8;
constexpr int kTileMaxRows = 7000;
constexpr int kTileMaxColumns = (1 << 26) - 4;

// In-plane part of a column's rays: origin s, direction r on axes 0 and 1 (the
// arithmetic of ray_line, in which dv_0 = dv_1 = 0 adds nothing) and the
// driving axis.
struct Column {
  double s0, s1, r0, r1;
  int m;
};
GJP_HD Column column_line(const double* __restrict__ v, bool cone, double u) {
  Column c;
  const double d0 = v[3] + u * v[6], d1 = v[4] + u * v[7];
  if (cone) {
    c.s0 = v[0];
    c.s1 = v[1];
    c.r0 = d0 - v[0];
    c.r1 = d1 - v[1];
  } else {
    c.s0 = d0;
    c.s1 = d1;
    c.r0 = v[0];
    c.r1 = v[1];
  }
  c.m = fabs(c.r1) > fabs(c.r0) ? 1 : 0;
  return c;
}

// What a tile (planes pm0 .. of axis m, rows ra0 .. of the other one, zt voxels from z0
// on along axis 2) needs of a view: columns whose in-plane line can come within a voxel
// of it on its planes, rows within a voxel of it along axis 2, counted from the
// detector's other end if dv points down (v0, rows as real numbers), and the ray spacings
// there; any: one of the columns is driven by axis m.
struct TileWindow {
  int ulo, uhi;
  double v0, rows, bmin, bmax;
  bool any;
};
GJP_HD TileWindow tile_window(const double* __restrict__ v, const float* __restrict__ Q, bool cone,
                              int n_u, int n_v, int m, int pm0, int ra0, int z0, int zt) {
  TileWindow w;
  float umin = 3.0e38f, umax = -3.0e38f;
#pragma unroll 1
  for (int k = 0; k < 4; ++k) {
    const float fp = (float)((k & 1) ? pm0 + kTileEdge - 1 : pm0);
    const float fr = (k & 2) ? (float)(ra0 + kTileEdge) + 0.01f : (float)ra0 - 1.01f;
    const float qx = m == 0 ? fp : fr, qy = m == 0 ? fr : fp;
    const float un = __builtin_fmaf(Q[0], qx, __builtin_fmaf(Q[1], qy, Q[3]));
    const float d = __builtin_fmaf(Q[8], qx, __builtin_fmaf(Q[9], qy, Q[11]));
    const float uu = un / d;
    umin = fminf(umin, uu);
    umax = fmaxf(umax, uu);
  }
  w.ulo = (int)ceilf(fminf(fmaxf(umin - 0.05f, 0.0f), (float)n_u));
  w.uhi = (int)floorf(fmaxf(fminf(umax + 0.05f, (float)(n_u - 1)), -1.0f));
  // rows: extremes at the corners (the row through a point of a plane is linear in u,
  // and monotone in the plane)
  const bool flip = v[11] < 0.0;
  double vmin = 1.0e300, vmax = -1.0e300;
  w.bmin = 1.0e300;
  w.bmax = 0.0;
  w.any = false;
#pragma unroll 1
  for (int k = 0; k < 4; ++k) {
    const double u = (double)((k & 1) ? w.uhi : w.ulo);
    const Column col = column_line(v, cone, u);
    w.any = w.any || col.m == m;
    const double sm = m == 0 ? col.s0 : col.s1, rm = m == 0 ? col.r0 : col.r1;
    const double t = ((double)((k & 2) ? pm0 + kTileEdge - 1 : pm0) - sm) / rm;
    const double d2 = v[5] + u * v[8] + (flip ? (double)(n_v - 1) * v[11] : 0.0);
    const double A = cone ? v[2] + t * (d2 - v[2]) : d2 + t * v[2];
    const double B = fabs(cone ? t * v[11] : v[11]);
    vmin = fmin(vmin, ((double)z0 - 1.01 - A) / B);
    vmax = fmax(vmax, ((double)(z0 + zt) + 0.01 - A) / B);
    w.bmin = fmin(w.bmin, B);
    w.bmax = fmax(w.bmax, B);
  }
  w.v0 = floor(vmin - 0.02);
  w.rows = ceil(vmax + 0.02) - w.v0 + 1.0;
  return w;
}

}  // namespace gjp

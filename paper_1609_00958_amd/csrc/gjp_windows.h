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

}  // namespace gjp

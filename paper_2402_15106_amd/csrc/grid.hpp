// The radius graph's uniform grid: box of the points, choice of the cells, and
// the cell of a point.  Host and device, so that the choice can be checked
// without a GPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>

namespace dsmp {

struct GridParams {
  float lo[3];
  int dims[3];
  int ncell;
  double inv_c;   // 1 / cell width
};

// Adds coordinate v to the extent [lo, hi].  Infinite and NaN coordinates are
// left out: no finite radius reaches such a point, and in the box they would
// leave a grid of one cell, or of no finite width.
__host__ __device__ __forceinline__ void box_add(float& lo, float& hi, float v) {
  if (!(fabsf(v) < INFINITY)) return;
  lo = fminf(lo, v);
  hi = fmaxf(hi, v);
}

// Grid of the box [lo, hi] (box_add's: finite, or lo > hi where it got no
// coordinate).  Cells are at least r*(1 + 2^-10) wide, so two points that pass
// the float32 radius test always sit in the same or adjacent cells (cell
// coordinates are formed in double, see cell_coord); the grid is coarsened by
// doubling until it has at most `cap` >= 1 cells.  That ends: extents of at most
// 2^129 against widths of 1e-30 and more are one cell after 229 doublings.  A
// radius whose float32 square overflows passes every distance, also infinite
// ones, and takes one cell.
__host__ __device__ __forceinline__ GridParams choose_grid(float lo[3], float hi[3], int D, float r, int64_t cap) {
  for (int a = D; a < 3; ++a) { lo[a] = 0.0f; hi[a] = 0.0f; }
  for (int a = 0; a < 3; ++a)
    if (!(hi[a] >= lo[a])) { lo[a] = 0.0f; hi[a] = 0.0f; }   // empty input
  double c = r * r < INFINITY ? (double)r * (1.0 + 1.0 / 1024.0) : (double)INFINITY;
  if (!(c > 1e-30)) c = 1e-30;
  double dims[3];
  for (;;) {
    double cells = 1.0;
    for (int a = 0; a < 3; ++a) {
      dims[a] = floor(((double)hi[a] - (double)lo[a]) / c) + 1.0;
      cells *= dims[a];
    }
    if (!(cells > (double)cap)) break;
    c *= 2.0;
  }
  GridParams g;
  for (int a = 0; a < 3; ++a) { g.lo[a] = lo[a]; g.dims[a] = (int)dims[a]; }
  g.inv_c = 1.0 / c;
  g.ncell = g.dims[0] * g.dims[1] * g.dims[2];
  return g;
}

// Cell of coordinate v, in double: v - lo is exact there and the product
// with 1/c is within 2^-52 of the cell coordinate, so the cell margin of
// 2^-10 covers the rounding however many cells an axis has (in float32 the
// worst-case error grows with the coordinate and reaches the margin at a few
// thousand cells on an axis, which a long, thin point set can have).
// Coordinates off the box, infinite ones too, fall in its first or last cell,
// NaN in the first: clamped before the conversion to int, which has no result
// for them.
__host__ __device__ __forceinline__ int cell_coord(float v, float lo, double inv_c, int dim) {
  const double t = ((double)v - (double)lo) * inv_c;
  return (int)fmin(fmax(t, 0.0), (double)(dim - 1));
}

__host__ __device__ __forceinline__ uint32_t cell_of(float3 p, const GridParams& g, int D) {
  const int cx = cell_coord(p.x, g.lo[0], g.inv_c, g.dims[0]);
  const int cy = cell_coord(p.y, g.lo[1], g.inv_c, g.dims[1]);
  const int cz = D == 3 ? cell_coord(p.z, g.lo[2], g.inv_c, g.dims[2]) : 0;
  return (uint32_t)(cx + g.dims[0] * (cy + g.dims[1] * cz));
}

}  // namespace dsmp

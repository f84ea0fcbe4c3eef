// Host run of the radius graph's grid (grid.hpp): every choice ends, its cells
// fit the table, and any two points that pass the float32 radius test lie in
// the same or adjacent cells.  Reads cases "D r cap n x y [z] ..." from stdin;
// prints "ncell pairs apart" per case.
#include <stdio.h>
#include <math.h>
#include <vector>
#include "../../paper_2402_15106_amd/csrc/grid.hpp"

using namespace dsmp;

int main() {
  int D, n;
  long long cap;
  float r;
  while (scanf("%d %f %lld %d", &D, &r, &cap, &n) == 4) {
    std::vector<float> p(3 * (size_t)n, 0.0f);
    for (int i = 0; i < n; ++i)
      for (int a = 0; a < D; ++a)
        if (scanf("%f", &p[3 * i + a]) != 1) return 1;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = 0; i < n; ++i)
      for (int a = 0; a < 3; ++a) box_add(lo[a], hi[a], p[3 * i + a]);
    const GridParams g = choose_grid(lo, hi, D, r, cap);
    if (g.ncell < 1 || g.ncell > cap) return 2;
    long pairs = 0, apart = 0;
    const float r2 = r * r;
    for (int i = 0; i < n; ++i) {
      if (cell_of(make_float3(p[3 * i], p[3 * i + 1], p[3 * i + 2]), g, D) >= (uint32_t)g.ncell) return 3;
      for (int j = 0; j < i; ++j) {
        volatile float d2 = 0.0f;
        bool near = true;
        for (int a = 0; a < D; ++a) {
          volatile float dx = p[3 * j + a] - p[3 * i + a], sq = dx * dx;
          d2 = a == 0 ? sq : d2 + sq;
          const int ci = cell_coord(p[3 * i + a], g.lo[a], g.inv_c, g.dims[a]);
          const int cj = cell_coord(p[3 * j + a], g.lo[a], g.inv_c, g.dims[a]);
          near = near && abs(ci - cj) <= 1;
        }
        if (!(d2 <= r2)) continue;
        ++pairs;
        apart += !near;
      }
    }
    printf("%d %ld %ld\n", g.ncell, pairs, apart);
    fflush(stdout);
  }
  return 0;
}

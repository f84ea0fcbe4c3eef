// The forms the library's backward takes: reads "dtype d n E" lines, prints
// "dz_with_m fused" for each (aggregate form, the shapes of width d).
#include <stdio.h>
#include "../../paper_2402_15106_amd/csrc/nnconv.hpp"

int main() {
  int dtype, d;
  long long n, E;
  while (scanf("%d %d %lld %lld", &dtype, &d, &n, &E) == 4) {
    const dsmp_layer_desc desc{3, d, 2 * d, 2 * d, dtype, DSMP_ACT_IDENTITY, 1, DSMP_ATTR_CONCAT};
    printf("%d %d\n", (int)dsmp::dz_with_m(desc, true, n, E), (int)dsmp::fused_edge_grads(desc, n, E));
  }
  return 0;
}

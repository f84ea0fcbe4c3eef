// launch_outer_sum (bf16, d = 64 and 32) with an edge order: refused on the
// host, before anything is launched.  Prints the status and the message.
#include <stdio.h>
#include "../../paper_2402_15106_amd/csrc/nnconv.hpp"

int main() {
  for (int d = 64; d >= 32; d /= 2) {
    dsmp_handle h;
    dsmp_layer_desc desc{2, d, 2 * d, 2 * d, DSMP_BF16, DSMP_ACT_IDENTITY, 1, DSMP_ATTR_CONCAT};
    int32_t order[1] = {0};
    const dsmp_status st = dsmp::launch_outer_sum(&h, desc, 1, 1, order, order, order, nullptr, nullptr, nullptr);
    printf("%d %s\n", (int)st, h.err.c_str());
  }
  return 0;
}

// Host check of the dispatch rules (dispatch.h): reads lines of a word and five
// numbers and prints what each shape takes. Built host-only by
// tests/test_dispatch_host.py.
//   score <stride> <causal> <heads> <blocks> <compute units>     rows of the tile
//   attn <query heads> <kv heads> <blocks> <dense> <compute units>
//     2 for 32-query workgroups, else 1 for query block first (causal), else 0
#include <cstdio>
#include <cstring>

#include "dispatch.h"

using namespace xattn;

int main() {
  char what[16];
  int a, b, c, d, e;
  while (std::scanf("%15s %d %d %d %d %d", what, &a, &b, &c, &d, &e) == 6) {
    if (std::strcmp(what, "score") == 0) {
      std::printf("%d\n", score_tile_rows(c, d * kBlock / a, a, b != 0, e));
    } else if (std::strcmp(what, "attn") == 0) {
      const size_t kv_bytes = (size_t)4 * b * c * kBlock * kHeadDim;
      std::printf("%d\n", attn_small(a * c, c, e) ? 2 : attn_by_block(true, d != 0, kv_bytes, a * c, a / b));
    } else {
      return 1;
    }
  }
  return 0;
}

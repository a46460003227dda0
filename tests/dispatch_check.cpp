// Host check of the dispatch rules (dispatch.h): reads "score <stride> <causal>
// <heads> <blocks> <compute units>" lines and prints the rows of the tile that
// each shape takes. Built host-only by tests/test_dispatch_host.py.
#include <cstdio>
#include <cstring>

#include "dispatch.h"

using namespace xattn;

int main() {
  char what[16];
  int a, b, c, d, e;
  while (std::scanf("%15s %d %d %d %d %d", what, &a, &b, &c, &d, &e) == 6) {
    if (std::strcmp(what, "score") != 0) return 1;
    std::printf("%d\n", score_tile_rows(c, d * kBlock / a, a, b != 0, e));
  }
  return 0;
}

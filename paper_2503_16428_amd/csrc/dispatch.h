// Which kernel a shape takes: the rules, as functions of the shape and the
// number of compute units that the host can call (and tests check).
#pragma once

#include "common.h"
#include "score_rows.h"

namespace xattn {

__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// ---- scoring

constexpr int kTileMax = 256;  // reduced rows and columns of score_partials' tiles
constexpr int kChunk = 64;     // reduced-K chunk per pipeline stage (128-byte rows)

// Tiles of a head: 256 x 256, and kTsub columns x RT rows (score_partials_small;
// row tile rt has (rt RT) / kTsub + 1 column tiles when causal).
inline int large_tiles(bool causal, int NR) {
  const int T = ceil_div(NR, kTileMax);
  return causal ? T * (T + 1) / 2 : T * T;
}
inline int small_tiles(int RT, bool causal, int NR) {
  const int nrt = ceil_div(NR, RT), k = kTsub / RT, nct = ceil_div(NR, kTsub);
  if (!causal) return nrt * nct;
  const int g = (nrt - 1) / k;
  return k * (g * (g + 1) / 2) + (nrt - g * k) * (g + 1);
}

// Rows of the scoring's tiles, 256, 128, 64 or 32: those whose rounds over the
// chip (one workgroup per CU) cost least. A round takes a chunk's time (1.1 us
// per 64-deep chunk of 256 x 256, 0.52 of 128 x 128, 0.42 of 128 x 64, 0.30 of
// 128 x 32: a smaller tile moves more bytes per product but is done sooner) for
// each chunk, and its start and epilogue (8 / 3.6 / 2.5 / 1.8 us), measured
// with every CU busy; the first with 32x32x16 MFMAs, and any value from 1.04 to
// 1.10 gives the same choices at the shapes below. Small tiles win where the
// 256 x 256 ones would leave CUs idle, in a first round or in a second one, or
// be mostly edge. Measured with every tile at 983 shapes (all strides, 1 to 64
// heads, 2 to 256 blocks, causal and not; xattn_score): the choice is the
// fastest or within 4 % of it but at six shapes, where 256 x 256 would be 1.5
// to 2.6 us (5 to 9 %) faster. In 256 / 128 / 64 / 32 rows, causal: 4736
// tokens, one head, S = 8: 28 / 17 / 16 / 16 us; 16 heads, S = 16: 45 / 24 / 19
// / 26; 8K, 32 heads, S = 16: 48 / 44 / 46 / 56; 6400 tokens, 32 heads, S = 8
// (320 large tiles): 56 / 52 / 61 / 76; 8K, 24 heads (240): 37 / 53 / 64 / 89;
// 32 heads (320): 58 / 65 / 80 / 113.
inline int score_tile_rows(int heads, int NR, int stride, bool causal, int wgs) {
  const long long nch = stride * kHeadDim / kChunk;
  const int rows[4] = {kTileMax, 128, 64, 32};
  const long long chunk[4] = {110, 52, 42, 30}, ends[4] = {800, 360, 250, 180};  // 10 ns
  int best = 0;
  long long least = 0;
  for (int i = 0; i < 4; ++i) {
    const long long per_head = i == 0 ? large_tiles(causal, NR) : small_tiles(rows[i], causal, NR);
    const long long cost = (heads * per_head + wgs - 1) / wgs * (chunk[i] * nch + ends[i]);
    if (i == 0 || cost < least) {
      best = i;
      least = cost;
    }
  }
  return rows[best];
}

}  // namespace xattn

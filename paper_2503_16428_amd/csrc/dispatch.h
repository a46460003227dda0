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

// ---- attention

// 32-query workgroups (attn_small_kernel), four per query block, one per CU:
// while they fit the chip once, or twice where rows are long. Measured against
// the 128-query kernel (us, 256 CUs, 3 to 50 % of the blocks and dense):
//   once (up to 64 query blocks), never slower in 11 shapes, causal and not:
//   one head of 4K, 50 %, 43 -> 24, dense 61 -> 30; 8 heads of 768 tokens,
//   dense, 17.4 -> 12.1; one head of 8K, 15 %, 31.5 -> 19.3, dense 115 -> 55;
//   twice: 2 heads of 6K, 20 %, 36 -> 23; one head of 16K, 20 %, 67 -> 44,
//   dense 225 -> 130, bidirectional 81 -> 74 and 247 -> 228. Faster from lists
//   of 6 % on; at 3 % one head of 16K 24.9 -> 22.5 and, bidirectional, 26.7 ->
//   28.6, at 2 blocks a row 13.4 -> 16.1;
//   twice with shorter rows they lose where rows are alike: 8 heads of 2K,
//   bidirectional, dense, 36 -> 40, 16 heads of 1K 22 -> 27;
//   three times: one head of 20K, bidirectional, dense, 294 -> 370.
// Dense and listed calls choose alike, so that dense and full lists give the
// same bits.
inline bool attn_small(int n_work, int NB, int cus) {
  return 4ll * n_work <= cus || (2ll * n_work <= cus && NB >= 48);
}

// Work order of attn_kernel: query block first, then kv head, where rows differ
// in length (causal) and all heads' K/V share the caches; kv head after kv
// head, the light rows of one head run beside the heavy rows of the next, and
// the last head's tail leaves CUs idle. Measured, us: dense, 4K, 32/8 heads 179
// -> 140, 16K, 24 heads 1663 -> 1395, 32K, 32/8 (128 MB of K/V) 7416 -> 7222;
// lists, groups of up to 4: 4K, 24/8 (768 rows) 94 -> 70, 8K, 32/8 (2048) 220
// -> 203, 16K, 32/8 (4000) 586 -> 581, 32K, 12/4 (3000) 505 -> 511, 16/16
// (4000) 721 -> 692; groups of 5 to 8: 4K, 28/4 (896) 94 -> 80, 8K, 28/4 (1792)
// 184 -> 176, 64/8 at 4K (2048) 188 -> 175, 16K, 16/2 (2000) 286 -> 286. Lists
// with more rows live off the cache of one group's K/V instead: 32K, 32/8
// (8000) 1351 -> 1389, 16K, 64/16 (8000) 1148 -> 1200, and for wide groups 16K,
// 28/4 (3500) 498 -> 507, 8K, 64/8 (4096) 409 -> 416.
inline bool attn_by_block(bool causal, bool dense, size_t kv_bytes, int n_work, int group) {
  if (!causal) return false;
  return dense ? kv_bytes <= ((size_t)128 << 20) : n_work <= (group <= 4 ? 4096 : 2048);
}

}  // namespace xattn

// Step 1: strided antidiagonal block scoring (XAttention Sec. 3.2, Algorithm 1).
//
// The reshapes of Algorithm 1 make reduced row R of Q~ the concatenation
// (along features) of query rows R*S + S-1, ..., R*S and reduced column c of
// K~ the concatenation of key rows c*S, ..., c*S + S-1, so
//   X[R][c] = q~_R . k~_c = sum_{t<S} q[R*S + S-1-t] . k[c*S + t],
// the sum over the antidiagonal of the S x S sub-block (R, c) of Q K^T.
// K~ is a plain view of K ([L/S][S*d], row c at K + c*S*d) and Q~ a view of Q
// with the S sub-rows reversed: no data is moved to build either.
//
// Kernel score_partials computes X^T = K~ Q~^T in 256 x 256 tiles on bf16
// MFMA (16x16x32, fp32 accumulate; 8 waves of 128 columns x 64 rows; 64-deep K chunks
// streamed by direct-to-LDS loads through a two-stage pipeline) and, in its
// epilogue, per reduced row R and 128-column sub-tile t: the sub-tile max m
// (log2 domain), l = sum exp2(x - m), and per key block j the partial mass
// sum_{c in j} exp2(x - m). Kernel score_finalize
// merges the tiles of each row (m_R = max_t m, l_R = sum_t l 2^(m - m_R)),
// normalises, and averages the B/S reduced rows of each query block.
#include <atomic>
#include <type_traits>
#include <utility>

#include "common.h"
#include "dispatch.h"
#include "score_rows.h"
#include "select_rows.h"

using namespace xattn;

namespace {

constexpr int TM = kTileMax;        // reduced rows (R) and columns (c) per workgroup tile
constexpr int TSUB = kTsub;         // column sub-tile owning one (m, l) pair per row
constexpr int KC = kChunk;          // reduced-K chunk per pipeline stage (128-byte rows)
constexpr int NSTAGE = 2;           // stages: one chunk computed while the next loads
constexpr int kThreads = 512;       // 8 waves: 2 (columns) x 4 (rows), 128 c x 64 R each
constexpr int kStage = TM * KC;     // bf16 elements of one operand in one stage
constexpr int kCPR = KC / 8;        // 16-byte chunks per LDS row
constexpr int kRowsPer256 = 128 / KC;  // LDS rows per 256-byte bank period
constexpr int kDmaRows = 512 / KC;  // rows one 1 KB direct-to-LDS instruction fills
constexpr int kDmaPerOp = 32 / kDmaRows;  // instructions per wave per operand per chunk
static_assert(NSTAGE * 2 * kStage * 2 <= 160 * 1024, "LDS budget");

__device__ __forceinline__ void tri_decode(int t, int& rt, int& ct) {
  int r = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while (r * (r + 1) / 2 > t) --r;
  while ((r + 1) * (r + 2) / 2 <= t) ++r;
  rt = r;
  ct = t - r * (r + 1) / 2;
}

// LDS rows hold KC bf16 (kCPR chunks of 16 B); chunk c of row r sits at
// position c ^ ((r / kRowsPer256) mod kCPR), so 16 consecutive rows read at
// one logical chunk hit 16 distinct bank groups.
__device__ __forceinline__ int swz_row(int r) { return (r / kRowsPer256) & (kCPR - 1); }

// Lane l < 32 returns a[l] + a[l + 32]; lane l >= 32 returns b[l - 32] + b[l]
// (one v_permlane32_swap exchanges the upper half of a with the lower half of
// b).
__device__ __forceinline__ float half_pair_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// The same between the 16-lane rows of a half: rows 0 and 2 return a summed
// over their half's two rows, rows 1 and 3 return b.
__device__ __forceinline__ float row_pair_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
// The lane's number, computed where it is called for: what depends on it would
// otherwise be kept over the main loop, in scratch memory, and each reload
// waits for every load and store in flight.
__device__ __forceinline__ int lane_anew() {
  uint32_t zero = 0;
  asm volatile("" : "+v"(zero));
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}
// Sum of x over lanes l, l ^ 16, l ^ 32, l ^ 48, in each of them.
__device__ __forceinline__ float quad_sum(float x) {
  const float z = half_pair_sum(x, x);
  return row_pair_sum(z, z);
}
__device__ __forceinline__ float quad_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x),
                                            __builtin_bit_cast(uint32_t, x), false, false);
  x = fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
  r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x),
                                       __builtin_bit_cast(uint32_t, x), false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]),
               __builtin_bit_cast(float, (uint32_t)r[1]));
}

// NRB = reduced rows (and columns) per 128-token block = 128 / S.
template <int NRB, bool CAUSAL>
__global__ __launch_bounds__(kThreads, 1) void score_partials(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int hq, int hkv, int L,
    int NR, int NB, int NT, int tiles_per_head, int n_work, float scale_log2,
    SubRowPairing pairing, float* __restrict__ part, float2* __restrict__ stats) {
  constexpr int S = kBlock / NRB;
  constexpr int KD = S * kHeadDim;  // reduced inner dimension S*d
  constexpr int NCH = KD / KC;      // >= 2 (S >= 1)
  // [operand A = K~ rows (c) | B = Q~ rows (R)][stage][256 rows x 64]: both
  // stages of an operand lie within the 64 KB that an LDS read's constant
  // offset reaches, so they share address registers
  __shared__ __attribute__((aligned(1024))) uint16_t lds[NSTAGE * 2 * kStage];

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wv & 1, wr = wv >> 1;

  // Persistent: each workgroup runs a sequence of tiles. Logical order
  // (kv head, row tile, column tile, query head in group); XCD x (blockIdx %
  // 8) takes one contiguous range of it, so the heads of a group that share
  // K~ rows run on one L2. While the last chunk of a tile is computed, the
  // first chunk of the next tile loads; its epilogue then overlaps that load.
  const int x8 = blockIdx.x % kNumXcd, k8 = blockIdx.x / kNumXcd;
  const int nper = gridDim.x / kNumXcd;  // workgroups per XCD (grid is a multiple of 8)
  const int per = n_work / kNumXcd, rem = n_work % kNumXcd;
  const int lo = x8 * per + (x8 < rem ? x8 : rem);
  const int cnt_x = per + (x8 < rem ? 1 : 0);
  const int G = hq / hkv;

  // The tile being loaded: its head, first reduced row / column, operand
  // bases (scalar) and this lane's load offsets. After a tile's last chunk
  // load it is switched to the next tile, whose first chunk then loads while
  // the finished tile (h_done, R0_done, c0_done) runs its epilogue.
  int th = 0, tR0 = 0, tc0 = 0;
  const uint16_t* tQh = q;
  const uint16_t* tKg = k;
  uint32_t offA[kDmaPerOp], offB[kDmaPerOp];
  auto load_tile = [&](int w) {
    const int hh = w % G;
    const int rest = w / G;
    const int tile = rest % tiles_per_head;
    const int gidx = rest / tiles_per_head;
    th = __builtin_amdgcn_readfirstlane((gidx / hkv) * hq + (gidx % hkv) * G + hh);
    int rt, ct;
    if (CAUSAL) {
      tri_decode(tile, rt, ct);
    } else {
      rt = tile / ceil_div(NR, TM);
      ct = tile % ceil_div(NR, TM);
    }
    tR0 = __builtin_amdgcn_readfirstlane(rt * TM);
    tc0 = __builtin_amdgcn_readfirstlane(ct * TM);
    tQh = q + (size_t)th * L * kHeadDim;
    tKg = k + (size_t)__builtin_amdgcn_readfirstlane(gidx) * L * kHeadDim;
    // direct-to-LDS staging: per stage each wave loads rows 32 wv .. +32 of
    // both operands, kDmaPerOp instructions (kDmaRows rows x 2 KC bytes)
    // each; rows beyond NR are clamped to NR - 1 (results masked / not stored)
    const int ln = lane_anew();
#pragma unroll
    for (int i = 0; i < kDmaPerOp; ++i) {
      const int r = 32 * wv + kDmaRows * i + ln / kCPR;
      const int c = (ln & (kCPR - 1)) ^ swz_row(r);
      const int ra = min(tc0 + r, NR - 1), rb = min(tR0 + r, NR - 1);
      offA[i] = (uint32_t)(((size_t)ra * KD + c * 8) * 2);
      offB[i] = (uint32_t)(((size_t)rb * S * kHeadDim + c * 8) * 2);
    }
  };

  const uint32_t lds0 = XATTN_LDS_ADDR(lds);
  // lane t holds the query sub-row paired with key sub-row t; read per chunk
  // with v_readlane (a table lookup in kernel-argument memory would put a
  // scalar load and its wait on every chunk's critical path)
  const int qsub_lane = pairing.q[lane < S ? lane : 0];
  // Load pair i (operand A = K~ rows, B = Q~ rows) of chunk ch of tile t into
  // stage ch % NSTAGE.
  auto dma_pair = [&](int ch, int i) __attribute__((always_inline)) {
    const int kap0 = ch * KC;
    const uint16_t* baseA = tKg + kap0;
    const uint16_t* baseB =  // a stride of 1 has one sub-row
        tQh + (S == 1 ? 0 : __builtin_amdgcn_readlane(qsub_lane, kap0 / kHeadDim) * kHeadDim) +
        kap0 % kHeadDim;
    const uint32_t st = lds0 + (uint32_t)((ch % NSTAGE) * kStage * 2);
    const uint32_t row_lds = (uint32_t)((32 * wv + kDmaRows * i) * KC * 2);
    dma16(baseA, offA[i], st + row_lds);
    dma16(baseB, offB[i], st + NSTAGE * kStage * 2 + row_lds);
  };

  // 16 x 16 tiles: acc[t][n] holds columns 16 t + 4 lg + [0, 4) of row 16 n + l16
  f32x4 acc[8][4];

  // Operand fragments of one 32-deep k-step: 8 of K~ (16 columns each), 4 of
  // Q~ (16 rows each); the K~ fragment of a slot is replaced as soon as its
  // four MFMAs have been issued, the Q~ fragments alternate between two sets.
  u32x4 fa[8], fb[2][4];
  // Diagonal tiles are computed in full (their masked half is ~2% of the MFMA
  // work of a causal layer); a per-MFMA skip would break the inner loop into
  // branches that serialise every LDS read with its MFMA.
  // LDS byte addresses of this lane's fragments, per k-step; stage, column and
  // row tile are constant offsets. The empty asm keeps the compiler from
  // splitting them into one address register per offset.
  const uint32_t xa = (uint32_t)swz_row(l16);  // swizzle of this lane's rows (multiples of 16 away)
  uint32_t ad_a[2], ad_b[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const uint32_t coff = ((4 * ks + lg) ^ xa) * 16;
    ad_a[ks] = lds0 + (128 * wc + l16) * (KC * 2) + coff;
    ad_b[ks] = lds0 + NSTAGE * kStage * 2 + (64 * wr + l16) * (KC * 2) + coff;
    asm volatile("" : "+v"(ad_a[ks]), "+v"(ad_b[ks]));
  }
  typedef const __attribute__((address_space(3))) u32x4* lds_frag;
  auto read_a = [&](int stage, int ks, int t) __attribute__((always_inline)) {
    fa[t] = *(lds_frag)(uintptr_t)(ad_a[ks] + (uint32_t)(stage * kStage * 2 + 16 * t * KC * 2));
  };
  auto read_b = [&](int stage, int ks, int n) __attribute__((always_inline)) {
    fb[ks][n] = *(lds_frag)(uintptr_t)(ad_b[ks] + (uint32_t)(stage * kStage * 2 + 16 * n * KC * 2));
  };
  // One chunk, already in LDS stage STAGE with its k-step 0 in fa, fb[0]: 16
  // steps of 4 MFMAs (one K~ fragment against the four Q~ ones). Steps 0-7
  // read k-step 1. Two steps later, when those reads are in registers, the
  // wave waits for its loads of the next chunk; the barrier makes everyone's
  // visible and ends all reads of this stage. The remaining steps read the
  // next chunk's k-step 0 and issue the loads of the chunk after it (load(i),
  // i < 4), so no wave starts a chunk without operands.
  // 16x16x32 MFMAs, not 32x32x16: with the accumulators in VGPRs and operands
  // that change, the latter sustain 1.65 PFLOP/s on zeros and 1.29 on normal
  // data (2 waves per SIMD, no memory traffic), these 2.45 and 2.05; at the
  // power limit the shader clock rises from 1.45 to 1.62 GHz. xattn_score with
  // waits at the chunk's start and 32x32x16, with these waits, with both
  // (finalize included): 128K, 32/8 heads, S = 16: 4.05, 3.99, 3.72 ms; 64K,
  // S = 4: 4.71, 4.36, 4.10 ms; 32K, S = 8: 0.571, 0.548, 0.514 ms.
  auto chunk = [&](auto stage_tag, bool zero, bool read_next, auto load) __attribute__((always_inline)) {
    constexpr int STAGE = decltype(stage_tag)::value;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int t = s & 7, ks = s >> 3;
      if (s == 10) {
        wait_vmcnt<0>();
        barrier_nofence();
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // back and forth, so that one operand stays the same (0.7 % faster)
        const int n = s & 1 ? 3 - i : i;
        acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            as_bf16x8(fa[t]), as_bf16x8(fb[ks][n]), zero && ks == 0 ? f32x4{} : acc[t][n], 0, 0, 0);
      }
      if (s < 8) {
        read_a(STAGE, 1, t);
        if (s >= 4) read_b(STAGE, 1, s - 4);
      }
      if (s >= 10) {  // the next chunk's k-step 0: Q~ and the first K~ fragments first
        constexpr int N = STAGE ^ 1;
        if (read_next) {
          if (s == 10) { read_a(N, 0, 0); read_b(N, 0, 0); }
          if (s == 11) { read_b(N, 0, 1); read_b(N, 0, 2); }
          if (s == 12) { read_b(N, 0, 3); read_a(N, 0, 1); }
          if (s == 13) { read_a(N, 0, 2); read_a(N, 0, 3); }
          if (s == 14) { read_a(N, 0, 4); read_a(N, 0, 5); }
          if (s == 15) { read_a(N, 0, 6); read_a(N, 0, 7); }
        }
        if (s == 15 || s % 2 == 0) load(s == 15 ? 3 : (s - 10) / 2);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  static_assert(KC == 64 && kDmaPerOp == 4 && NSTAGE == 2, "the chunk's two k-steps, four loads");

  auto epilogue = [&](const int h, const int R0, const int c0) __attribute__((always_inline)) {
    // ---- epilogue per 16-row slab n: this lane owns row R and 32 of the wave's
    // 128 columns; the lanes 16, 32 and 48 away own the others.
    const int csub = c0 + 128 * wc;  // first column of this wave's sub-tile
    const int tsub_idx = csub / TSUB;
    const int j0 = csub / NRB;
    const int ln = lane_anew(), l16 = ln & 15, lg = ln >> 4;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int Rslab = R0 + 64 * wr + 16 * n;
      const int R = Rslab + l16;
      // Invalid columns (c > R when causal, c >= NR) occur only in sub-tiles
      // that reach past the slab's first row or the reduced length; the empty
      // asm keeps this uniform branch from becoming selects on every tile.
      if ((CAUSAL && csub + 127 > Rslab) || csub + 127 >= NR) {
        asm volatile("");
        // last valid column of this row, relative to the lane's first one
        const int last = (CAUSAL ? min(R, NR - 1) : NR - 1) - csub - 4 * lg;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (16 * t + e > last) acc[t][n][e] = -INFINITY;
        }
      }
      // max of the raw products (the scale is positive), then every term as
      // one fma inside the exponential: p = 2^(x scale - m)
      float mloc = -INFINITY;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
#pragma unroll
        for (int e = 0; e < 4; ++e) mloc = fmaxf(mloc, acc[t][n][e]);
      }
      const float m = quad_max(mloc) * scale_log2;
      const float mref = (m == -INFINITY) ? 0.f : m;
      float gsum[8];  // this lane's 4 columns of tile t
      float lloc = 0.f;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = fast_exp2(fmaf(acc[t][n][e], scale_log2, -mref));
          if constexpr (NRB == 2) acc[t][n][e] = p;
          sum += p;
        }
        gsum[t] = sum;
        lloc += sum;
      }
      const float l = quad_sum(lloc);
      const bool rvalid = R < NR;
      // part is [head][query block][key block][row in block] (causal: key
      // blocks <= the query block only, rows packed as a triangle): what the
      // finalize workgroup of one query block reads is one contiguous slab.
      const int Rv = rvalid ? R : 0;
      const int qb = Rv / NRB;
      float* pcol = part + part_row(h, qb, NB, CAUSAL) * NRB + (Rv % NRB);
      // key block j of this row is stored if it exists and, when causal, is
      // not above the diagonal (those are fully masked and have no slot)
      auto put = [&](int j, float v) {
        if (rvalid && j < NB && (!CAUSAL || j <= qb)) pcol[(size_t)j * NRB] = v;
      };
      // A lane ends up with the totals that it stores: of four values summed
      // over the four lanes, lane group lg takes the lg-th.
      auto quad_of = [&](float v0, float v1, float v2, float v3) {
        return row_pair_sum(half_pair_sum(v0, v2), half_pair_sum(v1, v3));
      };
      if constexpr (NRB == 128) {
        if (lg == 0) put(j0, l);
      } else if constexpr (NRB == 64) {
        const float z = half_pair_sum(gsum[0] + gsum[1] + gsum[2] + gsum[3],
                                      gsum[4] + gsum[5] + gsum[6] + gsum[7]);
        const float tot = row_pair_sum(z, z);
        if ((lg & 1) == 0) put(j0 + (lg >> 1), tot);
      } else if constexpr (NRB == 32) {
        put(j0 + lg, quad_of(gsum[0] + gsum[1], gsum[2] + gsum[3], gsum[4] + gsum[5],
                             gsum[6] + gsum[7]));
      } else if constexpr (NRB == 16) {
#pragma unroll
        for (int u = 0; u < 8; u += 4)
          put(j0 + u + lg, quad_of(gsum[u], gsum[u + 1], gsum[u + 2], gsum[u + 3]));
      } else if constexpr (NRB == 8) {  // a tile's columns 0-7 are lane groups 0 and 1
#pragma unroll
        for (int t = 0; t < 8; t += 2)
          put(j0 + 2 * (t + (lg & 1)) + (lg >> 1), row_pair_sum(gsum[t], gsum[t + 1]));
      } else if constexpr (NRB == 4) {  // this lane's 4 columns of a tile are one block
#pragma unroll
        for (int t = 0; t < 8; ++t) put(j0 + 4 * t + lg, gsum[t]);
      } else {  // NRB == 2: they are two
        static_assert(NRB == 2, "stride must divide the block");
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          put(j0 + 8 * t + 2 * lg, acc[t][n][0] + acc[t][n][1]);
          put(j0 + 8 * t + 2 * lg + 1, acc[t][n][2] + acc[t][n][3]);
        }
      }
      // causal: a sub-tile starting after the row has no stats slot (all its
      // columns are masked for that row)
      if (rvalid && lg == 0 && tsub_idx < NT && (!CAUSAL || R >= tsub_idx * TSUB))
        stats[stats_at(h, tsub_idx, R, NR, NT, CAUSAL)] = make_float2(m, l);
    }
  };

  if (cnt_x <= k8) return;  // no tile for this workgroup (uniform)
  load_tile(lo + k8);
#pragma unroll
  for (int i = 0; i < kDmaPerOp; ++i) dma_pair(0, i);
#pragma unroll
  for (int i = 0; i < kDmaPerOp; ++i) dma_pair(1, i);
  wait_vmcnt<2 * kDmaPerOp>();  // chunk 0 has landed
  barrier_nofence();
  // k-step 0 of a tile (not before the epilogue: its registers are needed there)
  auto read_first = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < 4; ++n) read_b(0, 0, n);
#pragma unroll
    for (int t = 0; t < 8; ++t) read_a(0, 0, t);
  };
  read_first();
  using Even = std::integral_constant<int, 0>;
  using Odd = std::integral_constant<int, 1>;
  for (int it = k8; it < cnt_x; it += nper) {
    // Chunks in pairs (stage 0, stage 1). The last pair switches to the next
    // tile before it issues its first loads: that tile's chunks 0 and 1 are
    // then loaded before the epilogue. After the last tile the same tile's
    // chunks are loaded again (in bounds, never used).
    const int h_done = th, R0_done = tR0, c0_done = tc0;
    auto pair = [&](int ch, bool zero) __attribute__((always_inline)) {
      chunk(Even{}, zero, true, [&](int i) { dma_pair(ch + 2, i); });
      chunk(Odd{}, false, true, [&](int i) { dma_pair(ch + 3, i); });
    };
    // A loop of one pass: as straight code 2 and 4 chunks need more registers
    // than there are, and each reload waits for every load and store in flight
    // (S = 1, causal, four registers: 32K tokens, 2 heads 565 -> 540 us).
    auto in_loop = [](auto f) __attribute__((always_inline)) {
      int once = 1;
      asm volatile("" : "+s"(once));
#pragma unroll 1
      for (int i = 0; i < once; ++i) f();
    };
    if constexpr (NCH == 4) in_loop([&]() __attribute__((always_inline)) { pair(0, true); });
    else if constexpr (NCH > 2) pair(0, true);
#pragma unroll 1
    for (int ch = 2; ch + 2 < NCH; ch += 2) pair(ch, false);
    if (it + nper < cnt_x) load_tile(lo + it + nper);
    auto last_pair = [&]() __attribute__((always_inline)) {
      chunk(Even{}, NCH == 2, true, [&](int i) { dma_pair(0, i); });
      chunk(Odd{}, false, false, [&](int i) { dma_pair(1, i); });
    };
    if constexpr (NCH == 2) in_loop(last_pair);
    else last_pair();
    epilogue(h_done, R0_done, c0_done);
    read_first();
  }
  wait_vmcnt<0>();  // the last loads land before the LDS is released
}

// Small problems: the same partial sums in tiles of 128 columns (one sub-tile)
// x RT rows, one workgroup of 4 waves each. A few 256 x 256 tiles leave most
// CUs idle, and each is a serial chain of chunks as long as the load latency;
// these tiles are 4 to 16 times as many, and a ring of 4 to 6 LDS stages keeps
// 80 to 120 KB of loads in flight per CU (a chunk of a 128 x 32 tile takes
// 0.22 us alone, one of a 256 x 256 tile 1.05 us). The sums are those of
// score_partials in another order: 16 products an MFMA and not 32, and a row's
// columns over other lanes and waves. So a head's scores may differ in their
// last bits with the number of heads and blocks that choose the tile.
template <int RT>
struct SmallTile {
  static constexpr int kWc = RT >= 128 ? 2 : 4;        // waves along the columns
  static constexpr int kTn = TSUB / 32 / kWc;          // 32-column tiles per wave
  static constexpr int kRn = RT / 32 / (4 / kWc);      // 32-row tiles per wave
  static constexpr int kRows = TSUB + RT;              // LDS rows per stage (K~, then Q~)
  static constexpr int kIpw = kRows / kDmaRows / 4;    // load instructions per wave per chunk
  static constexpr int kStages = RT >= 128 ? 4 : 6;      // even; 120 - 144 KB of LDS
  static constexpr int kStageElems = kRows * KC;
};

// f(integral_constant<int, I>) for every I of the sequence, in order.
template <int... I, typename F>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}

template <int NRB, bool CAUSAL, int RT>
__global__ __launch_bounds__(256, 1) void score_partials_small(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int hq, int hkv, int L,
    int NR, int NB, int NT, int tiles_per_head, int n_work, float scale_log2,
    SubRowPairing pairing, float* __restrict__ part, float2* __restrict__ stats) {
  using T = SmallTile<RT>;
  constexpr int S = kBlock / NRB, KD = S * kHeadDim, NCH = KD / KC;
  constexpr int kAhead = NCH < T::kStages ? NCH : T::kStages;  // chunks in flight
  __shared__ __attribute__((aligned(1024))) uint16_t lds[T::kStages * T::kStageElems];
  __shared__ float red_m[4][RT], red_s[4][RT];

  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wv % T::kWc, wr = wv / T::kWc;

  const int x8 = blockIdx.x % kNumXcd, k8 = blockIdx.x / kNumXcd;
  const int per = n_work / kNumXcd, rem = n_work % kNumXcd;
  if (k8 >= per + (x8 < rem ? 1 : 0)) return;  // uniform
  const int w = x8 * per + (x8 < rem ? x8 : rem) + k8;
  const int G = hq / hkv;
  const int hh = w % G, rest = w / G;
  const int tile = rest % tiles_per_head, gidx = rest / tiles_per_head;
  const int h = __builtin_amdgcn_readfirstlane((gidx / hkv) * hq + (gidx % hkv) * G + hh);
  int rt, ct;
  if (CAUSAL) {
    constexpr int kk = TSUB / RT;
    int g, unused;
    tri_decode(tile / kk, g, unused);
    const int r = tile - kk * (g * (g + 1) / 2);
    rt = g * kk + r / (g + 1);
    ct = r % (g + 1);
  } else {
    rt = tile / NT;
    ct = tile % NT;
  }
  const int R0 = __builtin_amdgcn_readfirstlane(rt * RT);
  const int c0 = __builtin_amdgcn_readfirstlane(ct * TSUB);
  const uint16_t* Qh = q + (size_t)h * L * kHeadDim;
  const uint16_t* Kg = k + (size_t)__builtin_amdgcn_readfirstlane(gidx) * L * kHeadDim;

  // load i of this wave fills LDS rows kDmaRows (kIpw wv + i) .. of a stage;
  // rows beyond NR are clamped to NR - 1 (results masked / not stored)
  uint32_t off[T::kIpw];
#pragma unroll
  for (int i = 0; i < T::kIpw; ++i) {
    const int r = kDmaRows * (T::kIpw * wv + i) + lane / kCPR;
    const int c = (lane & (kCPR - 1)) ^ swz_row(r);
    const int src = r < TSUB ? min(c0 + r, NR - 1) : min(R0 + r - TSUB, NR - 1);
    off[i] = (uint32_t)(((size_t)src * KD + c * 8) * 2);
  }
  const uint32_t lds0 = XATTN_LDS_ADDR(lds);
  const int qsub_lane = pairing.q[lane < S ? lane : 0];
  auto load_chunk = [&](int ch) __attribute__((always_inline)) {
    const int kap0 = ch * KC;
    const uint16_t* baseA = Kg + kap0;
    const uint16_t* baseB =
        Qh + __builtin_amdgcn_readlane(qsub_lane, kap0 / kHeadDim) * kHeadDim + kap0 % kHeadDim;
    const uint32_t st = lds0 + (uint32_t)((ch % T::kStages) * T::kStageElems * 2);
#pragma unroll
    for (int i = 0; i < T::kIpw; ++i) {
      const int row = kDmaRows * (T::kIpw * wv + i);  // uniform
      dma16(row < TSUB ? baseA : baseB, off[i], st + (uint32_t)(row * KC * 2));
    }
  };

  f32x16 acc[T::kTn][T::kRn];
#pragma unroll
  for (int t = 0; t < T::kTn; ++t)
#pragma unroll
    for (int n = 0; n < T::kRn; ++n) acc[t][n] = f32x16{};
  const uint32_t xa = (uint32_t)swz_row(lr);
  struct Frags {  // operands of one chunk
    u32x4 a[KC / 16][T::kTn], b[KC / 16][T::kRn];
  };
  Frags f0, f1;
  auto read_chunk = [&](int ch, Frags& f) __attribute__((always_inline)) {
    const uint16_t* A = lds + (ch % T::kStages) * T::kStageElems;
    const uint16_t* Bm = A + TSUB * KC;
#pragma unroll
    for (int ks = 0; ks < KC / 16; ++ks) {
      const uint32_t coff = (uint32_t)((((2 * ks + lh) ^ xa)) << 3);
#pragma unroll
      for (int t = 0; t < T::kTn; ++t)
        f.a[ks][t] = *(const u32x4*)(A + (32 * (T::kTn * wc + t) + lr) * KC + coff);
#pragma unroll
      for (int n = 0; n < T::kRn; ++n)
        f.b[ks][n] = *(const u32x4*)(Bm + (32 * (T::kRn * wr + n) + lr) * KC + coff);
    }
  };
  auto mfma_chunk = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KC / 16; ++ks)
#pragma unroll
      for (int t = 0; t < T::kTn; ++t)
#pragma unroll
        for (int n = 0; n < T::kRn; ++n)
          acc[t][n] = mfma32(as_bf16x8(f.a[ks][t]), as_bf16x8(f.b[ks][n]), acc[t][n]);
  };

  for (int ch = 0; ch < kAhead; ++ch) load_chunk(ch);
  wait_vmcnt<(kAhead - 1) * T::kIpw>();
  barrier_nofence();
  read_chunk(0, f0);
  // Step ch: chunk ch + 1 has landed for this wave; the barrier makes
  // everyone's visible and ends every wave's reads of chunk ch, whose stage
  // receives chunk ch + kAhead; chunk ch + 1 is read while chunk ch's MFMAs run.
  auto step = [&](int ch, const Frags& f, Frags& fn) __attribute__((always_inline)) {
    wait_vmcnt<(kAhead - 2) * T::kIpw>();
    barrier_nofence();
    load_chunk(ch + kAhead);
    read_chunk(ch + 1, fn);
    mfma_chunk(f);
  };
  static_assert(kAhead % 2 == 0 && NCH % 2 == 0, "steps come in pairs");
#pragma unroll 1
  for (int ch = 0; ch < NCH - kAhead; ch += 2) {
    step(ch, f0, f1);
    step(ch + 1, f1, f0);
  }
  for_each_index(std::make_integer_sequence<int, kAhead>{}, [&](auto i) {
    constexpr int I = decltype(i)::value;
    if constexpr (I + 1 < kAhead) {
      wait_vmcnt<(kAhead - 2 - I) * T::kIpw>();
      barrier_nofence();
      read_chunk(NCH - kAhead + I + 1, I % 2 ? f0 : f1);
    }
    mfma_chunk(I % 2 ? f1 : f0);
  });

  // ---- epilogue: lane (lr, lh) holds, per 32 x 32 tile, row lr and columns
  // 8 g + 4 lh + [0, 4); a row's 128 columns span the kWc column waves.
  const int cw = 32 * T::kTn * wc;  // this wave's first column in the tile
#pragma unroll
  for (int n = 0; n < T::kRn; ++n) {
    const int rl = 32 * (T::kRn * wr + n) + lr;  // row in the tile
    const int R = R0 + rl;
    const int last = (CAUSAL ? min(R, NR - 1) : NR - 1) - c0 - cw - 4 * lh;
    if (last < 32 * T::kTn) {
#pragma unroll
      for (int t = 0; t < T::kTn; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * t + 8 * (r >> 2) + (r & 3) > last) acc[t][n][r] = -INFINITY;
    }
    float mloc = -INFINITY;
#pragma unroll
    for (int t = 0; t < T::kTn; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, acc[t][n][r]);
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
    if (lh == 0) red_m[wc][rl] = mloc;
  }
  __syncthreads();
  float m_row[T::kRn];
#pragma unroll
  for (int n = 0; n < T::kRn; ++n) {
    const int rl = 32 * (T::kRn * wr + n) + lr;
    const int R = R0 + rl;
    float m = red_m[0][rl];
#pragma unroll
    for (int u = 1; u < T::kWc; ++u) m = fmaxf(m, red_m[u][rl]);
    m *= scale_log2;
    m_row[n] = m;
    const float mref = (m == -INFINITY) ? 0.f : m;
    const bool rvalid = R < NR;
    const int Rv = rvalid ? R : 0;
    const int qb = Rv / NRB;
    float* pcol = part + part_row(h, qb, NB, CAUSAL) * NRB + (Rv % NRB);
    auto keep = [&](int j) { return rvalid && j < NB && (!CAUSAL || j <= qb); };
    float lloc = 0.f;
#pragma unroll
    for (int t = 0; t < T::kTn; ++t) {
      const int j0 = (c0 + cw + 32 * t) / NRB;
      float gsum[4];
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = fast_exp2(fmaf(acc[t][n][4 * g4 + e], scale_log2, -mref));
          acc[t][n][4 * g4 + e] = p;
          sum += p;
        }
        gsum[g4] = sum;
        lloc += sum;
      }
      if constexpr (NRB == 8) {  // group g is block g
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const float tot = half_pair_sum(gsum[x], gsum[x + 2]);
          const int j = j0 + 2 * lh + x;
          if (keep(j)) pcol[(size_t)j * NRB] = tot;
        }
      } else if constexpr (NRB == 16) {
        const float tot = half_pair_sum(gsum[0] + gsum[1], gsum[2] + gsum[3]);
        if (keep(j0 + lh)) pcol[(size_t)(j0 + lh) * NRB] = tot;
      } else if constexpr (NRB == 32) {
        const float s0 = gsum[0] + gsum[1] + gsum[2] + gsum[3];
        const float tot = half_pair_sum(s0, s0);
        if (lh == 0 && keep(j0)) pcol[(size_t)j0 * NRB] = tot;
      } else if constexpr (NRB == 4) {
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int j = j0 + 2 * g4 + lh;
          if (keep(j)) pcol[(size_t)j * NRB] = gsum[g4];
        }
      } else if constexpr (NRB == 2) {
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int j = j0 + 4 * g4 + 2 * lh;
          if (keep(j)) pcol[(size_t)j * NRB] = acc[t][n][4 * g4] + acc[t][n][4 * g4 + 1];
          if (keep(j + 1))
            pcol[(size_t)(j + 1) * NRB] = acc[t][n][4 * g4 + 2] + acc[t][n][4 * g4 + 3];
        }
      }
    }
    const float l = lloc + __shfl_xor(lloc, 32);
    if (lh == 0) red_s[wc][rl] = l;
  }
  __syncthreads();
  // row totals over the column waves; blocks wider than a wave's columns
  // (NRB = 64, 128) are sums of the same per-wave totals
  if (wc == 0 && lh == 0) {
#pragma unroll
    for (int n = 0; n < T::kRn; ++n) {
      const int rl = 32 * (T::kRn * wr + n) + lr;
      const int R = R0 + rl;
      float l = red_s[0][rl];
#pragma unroll
      for (int u = 1; u < T::kWc; ++u) l += red_s[u][rl];
      if (R < NR && (!CAUSAL || R >= c0))
        stats[stats_at(h, c0 / TSUB, R, NR, NT, CAUSAL)] = make_float2(m_row[n], l);
      if constexpr (NRB >= 64) {
        constexpr int kPer = NRB * T::kWc / TSUB;  // column waves per block
        if (R < NR) {
          const int qb = R / NRB;
          float* pcol = part + part_row(h, qb, NB, CAUSAL) * NRB + R % NRB;
#pragma unroll
          for (int x = 0; x < T::kWc / kPer; ++x) {
            const int j = c0 / NRB + x;
            float tot = 0.f;
#pragma unroll
            for (int u = 0; u < kPer; ++u) tot += red_s[x * kPer + u][rl];
            if (j < NB && (!CAUSAL || j <= qb)) pcol[(size_t)j * NRB] = tot;
          }
        }
      }
    }
  }
}

// One workgroup (4 waves) per (query head, query block) row: the row's
// scores from its partial sums and tile statistics (finalize_row).
template <bool CAUSAL, bool MANY>
__global__ __launch_bounds__(kFinThreads) void score_finalize(const float* __restrict__ part,
                                                              const float2* __restrict__ stats,
                                                              int NR, int NB, int NT, int nrb,
                                                              float* __restrict__ scores) {
  __shared__ FinalizeLds lds;
  const int h = blockIdx.x / NB, b = blockIdx.x % NB;
  finalize_row<CAUSAL, MANY>(part, stats, NR, NB, NT, nrb, h, b,
                             scores + ((size_t)h * NB + b) * NB, lds);
}

// The same, and the row's block list by wave 0 from the scores just written
// (they come back out of the L1 / L2 of the compute unit that wrote them):
// one launch and one pass less where the rows are few. NPL as in
// select_kernel.
template <int NPL, bool CAUSAL, bool MANY>
__global__ __launch_bounds__(kFinThreads) void score_finalize_select(
    const float* __restrict__ part, const float2* __restrict__ stats, int NR, int NB, int NT,
    int nrb, float tau, float* scores, int32_t* __restrict__ idx, int32_t* __restrict__ cnt) {
  __shared__ FinalizeLds lds;
  __shared__ uint32_t stage[64];
  const int h = blockIdx.x / NB, b = blockIdx.x % NB;
  const size_t row = (size_t)h * NB + b;
  finalize_row<CAUSAL, MANY>(part, stats, NR, NB, NT, nrb, h, b, scores + row * NB, lds);
  __syncthreads();
  if (threadIdx.x >= kWave) return;
  const int m = CAUSAL ? b + 1 : NB;
  select_row_sized<NPL, false>(scores + row * NB, m, tau, 0, threadIdx.x, idx + row * NB,
                               cnt + row, stage);
}

template <int NRB, bool CAUSAL, int RT>
hipError_t launch_small(const void* q, const void* k, const XattnShape& s,
                        const SubRowPairing& pr, float scale_log2, float* part, float* stats,
                        hipStream_t st) {
  const int NR = s.seq / (kBlock / NRB), tiles = small_tiles(RT, CAUSAL, NR);
  const int n_work = s.HQ() * tiles;
  hipLaunchKernelGGL((score_partials_small<NRB, CAUSAL, RT>),
                     dim3(ceil_div(n_work, kNumXcd) * kNumXcd), dim3(256), 0, st,
                     (const uint16_t*)q, (const uint16_t*)k, s.hq, s.hkv, s.seq, NR, s.NB(),
                     ceil_div(NR, TSUB), tiles, n_work, scale_log2, pr, part, (float2*)stats);
  return hipGetLastError();
}

template <int NRB, bool CAUSAL>
hipError_t launch_partials(const void* q, const void* k, const XattnShape& s,
                           const SubRowPairing& pr, float* part, float* stats, hipStream_t st) {
  const int S = kBlock / NRB, NR = s.seq / S, NB = s.NB(), NT = ceil_div(NR, TSUB);
  const int tiles = large_tiles(CAUSAL, NR);
  const int n_work = s.batch * s.hkv * tiles * (s.hq / s.hkv);
  const float scale_log2 = kLog2e / (sqrtf((float)kHeadDim) * (float)S);
  // one resident workgroup per CU (128 KB of LDS each), a multiple of 8
  const int wgs = compute_units();
  switch (score_tile_rows(s.HQ(), NR, S, CAUSAL, wgs)) {
    case 128: return launch_small<NRB, CAUSAL, 128>(q, k, s, pr, scale_log2, part, stats, st);
    case 64: return launch_small<NRB, CAUSAL, 64>(q, k, s, pr, scale_log2, part, stats, st);
    case 32: return launch_small<NRB, CAUSAL, 32>(q, k, s, pr, scale_log2, part, stats, st);
  }
  hipLaunchKernelGGL((score_partials<NRB, CAUSAL>), dim3(wgs), dim3(kThreads), 0, st,
                     (const uint16_t*)q, (const uint16_t*)k, s.hq, s.hkv, s.seq, NR, NB, NT,
                     tiles, n_work, scale_log2, pr, part, (float2*)stats);
  return hipGetLastError();
}

template <int NRB>
hipError_t launch_partials_c(const void* q, const void* k, const XattnShape& s,
                             const SubRowPairing& pr, float* part, float* stats, hipStream_t st) {
  return s.causal ? launch_partials<NRB, true>(q, k, s, pr, part, stats, st)
                  : launch_partials<NRB, false>(q, k, s, pr, part, stats, st);
}

}  // namespace

int compute_units() {
  static std::atomic<int> cached[64];  // static storage: starts at zero
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = 0;
  const bool cacheable = dev >= 0 && dev < 64;
  int n = cacheable ? cached[dev].load(std::memory_order_relaxed) : 0;
  if (n == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < kNumXcd)
      cus = 256;  // any multiple of 8 is a valid grid; this only sizes it
    n = cus / kNumXcd * kNumXcd;
    if (cacheable) cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

size_t score_scratch_bytes(const XattnShape& s, int stride) {
  const int NR = s.seq / stride, NB = s.NB(), NT = ceil_div(NR, TSUB);
  const size_t part = part_elems(s.HQ(), NB, kBlock / stride, s.causal) * sizeof(float);
  const size_t stats = (size_t)s.HQ() * stats_per_head(NR, NT, s.causal) * sizeof(float2);
  return ((part + 255) / 256) * 256 + stats;
}

ScoreScratch score_scratch_views(const XattnShape& s, int stride, void* scratch) {
  const size_t part_bytes =
      part_elems(s.HQ(), s.NB(), kBlock / stride, s.causal) * sizeof(float);
  ScoreScratch v;
  v.part = (float*)scratch;
  v.stats = (float*)((char*)scratch + ((part_bytes + 255) / 256) * 256);
  return v;
}

// The partial-sum kernel of xattn_score (the first of its two launches).
static hipError_t launch_score_partials(const void* q, const void* k, const XattnShape& s, int stride,
                                 const int32_t* qsub, void* scratch, hipStream_t st) {
  SubRowPairing pr;
  for (int t = 0; t < stride; ++t) pr.q[t] = qsub ? qsub[t] : stride - 1 - t;
  const ScoreScratch v = score_scratch_views(s, stride, scratch);
  switch (stride) {
    case 1: return launch_partials_c<128>(q, k, s, pr, v.part, v.stats, st);
    case 2: return launch_partials_c<64>(q, k, s, pr, v.part, v.stats, st);
    case 4: return launch_partials_c<32>(q, k, s, pr, v.part, v.stats, st);
    case 8: return launch_partials_c<16>(q, k, s, pr, v.part, v.stats, st);
    case 16: return launch_partials_c<8>(q, k, s, pr, v.part, v.stats, st);
    case 32: return launch_partials_c<4>(q, k, s, pr, v.part, v.stats, st);
    case 64: return launch_partials_c<2>(q, k, s, pr, v.part, v.stats, st);
    default: return hipErrorInvalidValue;
  }
}

template <int NPL, bool CAUSAL>
static void launch_finalize_select(const XattnShape& s, int stride, float tau, float* scores,
                                   int32_t* idx, int32_t* cnt, const ScoreScratch& v,
                                   hipStream_t st) {
  const int NR = s.seq / stride, NB = s.NB(), NT = ceil_div(NR, TSUB), nrb = kBlock / stride;
  auto kernel = nrb >= kFinalizeMany ? score_finalize_select<NPL, CAUSAL, true>
                                     : score_finalize_select<NPL, CAUSAL, false>;
  hipLaunchKernelGGL(kernel, dim3(s.HQ() * NB), dim3(kFinThreads), 0, st, v.part,
                     (const float2*)v.stats, NR, NB, NT, nrb, tau, scores, idx, cnt);
}

template <int NPL>
static void launch_finalize_select_c(const XattnShape& s, int stride, float tau, float* scores,
                                     int32_t* idx, int32_t* cnt, const ScoreScratch& v,
                                     hipStream_t st) {
  if (s.causal) launch_finalize_select<NPL, true>(s, stride, tau, scores, idx, cnt, v, st);
  else launch_finalize_select<NPL, false>(s, stride, tau, scores, idx, cnt, v, st);
}

// The launch it saves is 2 us of the layer: 1K tokens, one head, 27.8 -> 26.4
// us; 4K, one head, 35.6 -> 33.2 us; 8K, 32 heads (2048 rows, eight workgroups
// per compute unit at once) 290 -> 288 us. More rows gain nothing, and at 128K
// the three waves that wait for the search cost more than the launch.
bool score_select_fits(const XattnShape& s, float tau) {
  return tau < 1.f && s.NB() <= 256 && (long long)s.HQ() * s.NB() <= 2048;
}

hipError_t launch_score_select(const void* q, const void* k, const XattnShape& s, int stride,
                               float tau, float* scores, int32_t* idx, int32_t* cnt, void* scratch,
                               hipStream_t st) {
  hipError_t e = launch_score_partials(q, k, s, stride, nullptr, scratch, st);
  if (e != hipSuccess) return e;
  const ScoreScratch v = score_scratch_views(s, stride, scratch);
  if (s.NB() <= 64) launch_finalize_select_c<1>(s, stride, tau, scores, idx, cnt, v, st);
  else if (s.NB() <= 128) launch_finalize_select_c<2>(s, stride, tau, scores, idx, cnt, v, st);
  else launch_finalize_select_c<4>(s, stride, tau, scores, idx, cnt, v, st);
  return hipGetLastError();
}

hipError_t launch_score(const void* q, const void* k, const XattnShape& s, int stride,
                        const int32_t* qsub, float* scores, void* scratch, hipStream_t st) {
  hipError_t e = launch_score_partials(q, k, s, stride, qsub, scratch, st);
  if (e != hipSuccess) return e;
  const int NR = s.seq / stride, NB = s.NB(), NT = ceil_div(NR, TSUB);
  const int nrb = kBlock / stride;
  const ScoreScratch v = score_scratch_views(s, stride, scratch);
  const bool many = nrb >= kFinalizeMany;
  auto kernel = s.causal ? (many ? score_finalize<true, true> : score_finalize<true, false>)
                         : (many ? score_finalize<false, true> : score_finalize<false, false>);
  hipLaunchKernelGGL(kernel, dim3(s.HQ() * NB), dim3(kFinThreads), 0, st, v.part,
                     (const float2*)v.stats, NR, NB, NT, nrb, scores);
  return hipGetLastError();
}

// Scoring scratch layout and the per-row finalisation of the block scores
// (XAttention Sec. 3.2, Algorithm 1: reduced-row softmax, then the mean over
// each query block's B/S reduced rows of the per-key-block sums). Used by the
// scoring kernels (score.hip); the layout functions are host-callable too.
#pragma once

#include "common.h"

namespace xattn {

constexpr int kTsub = 128;      // reduced-column sub-tile owning one (max, sum) per row
constexpr int kFactorMax = 4096;  // (row, sub-tile) factors staged in LDS (16 KB) at a time
constexpr int kFinUnroll = 4;   // independent 16-byte partial-sum loads per thread
constexpr int kFinThreads = 256;
constexpr int kFinalizeMany = 64;  // reduced rows per block from which a thread has many sub-tiles

// Partial block masses, fp32: row (h, query block b) holds nrb floats per key
// block j, j < b + 1 when causal (the rows packed as a lower triangle), j <
// NB otherwise; element (h, b, j, r) at part_row(h, b) * nrb + j * nrb + r.
__host__ __device__ inline size_t part_row(int h, int b, int NB, bool causal) {
  return causal ? (size_t)h * ((size_t)NB * (NB + 1) / 2) + (size_t)b * (b + 1) / 2
                : ((size_t)h * NB + b) * NB;
}
__host__ __device__ inline size_t part_elems(int HQ, int NB, int nrb, bool causal) {
  return part_row(HQ, 0, NB, causal) * nrb;
}

// Row statistics (max, sum) per reduced row R and column sub-tile t, float2.
// Causal: only sub-tiles that start at or before the row (t * kTsub <= R)
// are kept, sub-tile t holding rows t * kTsub .. NR - 1; otherwise every
// (t, R). NT = ceil(NR / kTsub).
__host__ __device__ inline size_t stats_per_head(int NR, int NT, bool causal) {
  return causal ? (size_t)NT * NR - (size_t)kTsub * NT * (NT - 1) / 2 : (size_t)NT * NR;
}
__host__ __device__ inline size_t stats_at(int h, int t, int R, int NR, int NT, bool causal) {
  const size_t head = (size_t)h * stats_per_head(NR, NT, causal);
  return causal ? head + (size_t)t * NR - (size_t)kTsub * t * (t - 1) / 2 + (R - kTsub * t)
                : head + (size_t)t * NR + R;
}

// LDS of one finalisation (one workgroup of kFinThreads per row).
struct FinalizeLds {
  float red[2][kFinThreads];  // per wave (or pair of waves) and reduced row: max, sum
  float f[kFactorMax];        // f[(t - t0) * nrb + r]
};

// Block scores of row (h, b), nrb = B/S reduced rows R = b nrb + r and tn
// column sub-tiles per row:
//   m_R = max_t m[t][R],  l_R = sum_t l[t][R] 2^(m[t][R] - m_R),
//   f[r][t] = 2^(m[t][R] - m_R) / l_R,
//   out[j] = (1/nrb) sum_r part[j][r] f[r][t(j)]   for the candidates j,
//   out[j] = 0 for the other j < NB (causal: j > b).
// Thread i reads the stats of reduced row i mod nrb, sub-tiles i / nrb + u *
// (kFinThreads / nrb): the nrb rows of one sub-tile are adjacent in memory.
// The kFinThreads / nrb threads of a row are combined by shuffles inside a
// wave and through LDS across waves, in a fixed order. The
// factors are then staged kFactorMax at a time, and the part of the row's
// partial-sum slab [j][r] that they scale is streamed as float4 (or float2
// when nrb = 2), kFinUnroll loads in flight per thread; the nrb / 4 lanes of
// one block reduce with shuffles in a fixed order. Bound by the slab's bytes
// at every stride: at small strides a row has more factors than fit (S = 4:
// 4096 at 64K tokens, S = 1: 65536), and reading four stats and evaluating
// four exponentials per float4 instead took 0.420 ms at 64K, 32/8 heads,
// S = 4 (0.54 GB of partial sums). Called by all kFinThreads threads.
// MANY (nrb >= kFinalizeMany): a thread has up to 1024 sub-tiles, and one load
// at a time makes the row a chain of latencies; four are in flight
// (xattn_score, S = 1, causal: 32K tokens, 2 heads 540 -> 464 us; 4K, one head
// 24 -> 20 us). With smaller nrb it has few, and the unrolled loops cost 0.5
// us of 46 (8K, 32 heads, S = 16).
template <bool CAUSAL, bool MANY>
__device__ __forceinline__ void finalize_row(const float* __restrict__ part,
                                             const float2* __restrict__ stats, int NR, int NB,
                                             int NT, int nrb, int h, int b,
                                             float* __restrict__ out, FinalizeLds& L) {
  const int tid = threadIdx.x;
  const int ncand = CAUSAL ? b + 1 : NB;
  const int tn = CAUSAL ? (b * nrb) / kTsub + 1 : NT;  // sub-tiles of this row's stats
  const int R0 = b * nrb;
  const int r_own = tid % nrb, t_own = tid / nrb, tstep = kFinThreads / nrb;
  auto st = [&](int t) -> float2 {
    return stats[stats_at(h, t, R0 + r_own, NR, NT, CAUSAL)];
  };
  // the threads of one reduced row: lanes nrb apart in a wave (nrb < 64), then
  // the groups of max(nrb, 64) threads
  const int group = nrb > 64 ? nrb : 64, g_own = tid / group;
  const bool writes = tid % group < nrb;
  // f(t) for this thread's sub-tiles of t0 .. t1 - 1, in order
  auto each = [&](int t0, int t1, auto f) {
    if constexpr (MANY) {
#pragma unroll 4
      for (int t = t0 + t_own; t < t1; t += tstep) f(t);
    } else {
      for (int t = t0 + t_own; t < t1; t += tstep) f(t);
    }
  };
  float m = -INFINITY;
  each(0, tn, [&](int t) { m = fmaxf(m, st(t).x); });
  for (int off = 32; off >= nrb; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if (writes) L.red[0][g_own * nrb + r_own] = m;
  __syncthreads();
  m = L.red[0][r_own];
  for (int g = 1; g < kFinThreads / group; ++g) m = fmaxf(m, L.red[0][g * nrb + r_own]);
  float l = 0.f;
  each(0, tn, [&](int t) {
    const float2 v = st(t);
    l += v.y * fast_exp2(v.x - m);
  });
  for (int off = 32; off >= nrb; off >>= 1) l += __shfl_xor(l, off);
  if (writes) L.red[1][g_own * nrb + r_own] = l;
  __syncthreads();
  l = L.red[1][r_own];
  for (int g = 1; g < kFinThreads / group; ++g) l += L.red[1][g * nrb + r_own];
  const float il = 1.f / l;

  const float inv_nrb = 1.f / (float)nrb;
  const float* pb = part + part_row(h, b, NB, CAUSAL) * nrb;  // this row's slab [j][r]
  const int tchunk = kFactorMax / nrb;
  const int jper = kTsub / nrb;  // key blocks per sub-tile
  for (int t0 = 0; t0 < tn; t0 += tchunk) {
    const int t1 = min(t0 + tchunk, tn);
    each(t0, t1, [&](int t) { L.f[(t - t0) * nrb + r_own] = fast_exp2(st(t).x - m) * il; });
    __syncthreads();
    const int j_lo = t0 * jper, j_hi = min(t1 * jper, ncand);
    auto factor = [&](int r, int t) -> float { return L.f[(t - t0) * nrb + r]; };
    if (nrb >= 4) {
      // chunk q = 4 consecutive floats = rows 4 (q % (nrb/4)) .. +3 of block q / (nrb/4)
      const int cpb = nrb / 4;  // chunks (lanes) per block, a power of two <= 32
      const int nq = j_hi * cpb;
      const float4* p4 = (const float4*)pb;
      for (int q0 = j_lo * cpb; q0 < nq; q0 += kFinThreads * kFinUnroll) {
        float4 v[kFinUnroll];
#pragma unroll
        for (int u = 0; u < kFinUnroll; ++u) {
          const int q = q0 + kFinThreads * u + tid;
          v[u] = q < nq ? p4[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < kFinUnroll; ++u) {
          const int q = q0 + kFinThreads * u + tid;
          const int j = q / cpb, r0 = 4 * (q % cpb);
          const int t = (j * nrb) / kTsub;
          float acc = 0.f;
          if (q < nq)
            acc = v[u].x * factor(r0, t) + v[u].y * factor(r0 + 1, t) +
                  v[u].z * factor(r0 + 2, t) + v[u].w * factor(r0 + 3, t);
          for (int off = cpb / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
          if (q < nq && (q % cpb) == 0) out[j] = acc * inv_nrb;
        }
      }
    } else {  // nrb == 2: one float2 per block
      const float2* p2 = (const float2*)pb;
      for (int j0 = j_lo; j0 < j_hi; j0 += kFinThreads * kFinUnroll) {
        float2 v[kFinUnroll];
#pragma unroll
        for (int u = 0; u < kFinUnroll; ++u) {
          const int j = j0 + kFinThreads * u + tid;
          v[u] = j < j_hi ? p2[j] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < kFinUnroll; ++u) {
          const int j = j0 + kFinThreads * u + tid;
          if (j < j_hi) {
            const int t = (j * nrb) / kTsub;
            out[j] = (v[u].x * factor(0, t) + v[u].y * factor(1, t)) * inv_nrb;
          }
        }
      }
    }
    if (t1 < tn) __syncthreads();  // the factors are replaced
  }
  for (int j = ncand + tid; j < NB; j += kFinThreads) out[j] = 0.f;  // not candidates
}

}  // namespace xattn

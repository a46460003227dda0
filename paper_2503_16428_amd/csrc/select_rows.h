// Step 2: threshold block selection, find_blocks (XAttention Sec. 3.2).
//
// find_blocks asks for the smallest set of key blocks whose mass reaches tau.
// Masses are integers u_j = floor(clamp(score_j, 0, 1) * 2^32), so every sum
// below is exact and the result does not depend on summation order; the
// target is ceil(tau * T) with T the row total (one fp64 product).
//
// The same search serves the fixed-size selections of the Top-K / Top-Ratio
// ablation (Sec. 4.5, Table 6) with block counts instead of masses, and
// thresholds may differ per head (the consumer side of Sec. 3.3).
//
// One wave64 per (head, query block) row. Instead of sorting, the wave finds
// the mass v* of the last block the sorted prefix needs: the largest v with
// F(v) = sum_{u_j >= v} u_j >= target (F is non-increasing, so v* is one of
// the masses). The shortest prefix of the (u desc, j asc) order that reaches
// the target is then every block with u_j > v* plus the first
// ceil((target - F(v*+1)) / v*) blocks with u_j == v* in ascending j. Emitting
// in ascending j with ballot / mbcnt yields the index list already sorted.
//
// The search halves a bracket of values around v* geometrically (masses are
// spread over many binades) until at most 64 masses are left in it; these are
// gathered one per lane, and each lane adds up the ones not below its own.
// The kernel is bound by VALU work, not by memory: 64K tokens, 32 heads, the
// scores of clustered inputs, 50 us for a linear 33-step search over 64-bit
// masses (ten steps over every value), 18 us for this one; 128K 125 -> 43 us.
#pragma once

#include "common.h"

namespace xattn {

// Sum over the wave, returned uniform (in a scalar register): prefix sums
// inside each row of 16 lanes by DPP row shifts, then the four row totals.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  return __builtin_amdgcn_readlane(x, 15) + __builtin_amdgcn_readlane(x, 31) +
         __builtin_amdgcn_readlane(x, 47) + __builtin_amdgcn_readlane(x, 63);
}

// Exact wave sum of per-lane values below 2^42: the high and low 21-bit parts
// are summed separately (each total stays below 2^27).
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x) {
  const uint32_t hi = wave_sum_u32((uint32_t)(x >> 21));
  const uint32_t lo = wave_sum_u32((uint32_t)x & ((1u << 21) - 1u));
  return ((uint64_t)hi << 21) + lo;
}

// Number of lanes below this one in a ballot mask.
__device__ __forceinline__ uint32_t rank_in(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Max over the wave, returned uniform.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  auto mx = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  x = mx(x, __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false));
  return mx(mx(__builtin_amdgcn_readlane(x, 15), __builtin_amdgcn_readlane(x, 31)),
            mx(__builtin_amdgcn_readlane(x, 47), __builtin_amdgcn_readlane(x, 63)));
}

// One row with at most 64 NPL candidates; lane l holds j = l + 64 i. Every
// per-lane partial sum below is at most NPL * 2^32 <= 2^37.
//   COUNT = false (find_blocks): target = ceil(tau * T), F(v) = sum_{u >= v} u.
//   COUNT = true (Top-K / Top-Ratio): target = k, F(v) = #{u >= v}.
// A mass of 2^32 (a score of 1 or more) is held as 2^32 - 1, which no other
// score gives (the next one below 1 gives 2^32 - 256); `ones` of them are
// counted apart and added to every sum, as F is only taken at v <= hi.
// LEAST: the bracket starts at the row's least mass if that is higher.
template <int NPL, bool COUNT, bool LEAST = false>
__device__ __forceinline__ void select_row(const float* __restrict__ s, int m, float tau,
                                           int k, int lane, int32_t* __restrict__ out,
                                           int32_t* __restrict__ cnt_out,
                                           uint32_t* __restrict__ stage) {
  uint32_t u[NPL];
  uint64_t tl = 0;
  uint32_t top = 0, least = 0xFFFFFFFFu;
  uint32_t ones = 0;
  float v[NPL];
#pragma unroll
  for (int i = 0; i < NPL; ++i) v[i] = lane + 64 * i < m ? s[lane + 64 * i] : 0.f;
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    // NaN and negative -> 0; the product is exact and the conversion truncates
    const float x = v[i] > 0.f ? v[i] : 0.f;
    const bool one = x >= 1.f;
    ones += (uint32_t)__popcll(__ballot(one));
    u[i] = one ? 0xFFFFFFFFu : (uint32_t)(x * 4294967296.f);
    tl += u[i];
    top = u[i] > top ? u[i] : top;
    if (LEAST && lane + 64 * i < m) least = u[i] < least ? u[i] : least;
  }
  auto mass = [](uint32_t held) { return (uint64_t)held + (held == 0xFFFFFFFFu ? 1u : 0u); };
  uint64_t target, slack = 0;
  if constexpr (COUNT) {
    target = (uint64_t)k;  // 1 <= k < m
  } else {
    const uint64_t T = wave_sum_u64(tl) + ones;
    if (T == 0) {  // every candidate has zero mass: the first in (u desc, j asc) order is j = 0
      if (lane == 0) {
        out[0] = 0;
        *cnt_out = 1;
      }
      return;
    }
    const double prod = (double)tau * (double)T;
    target = (uint64_t)ceil(prod);
    slack = T - target;  // tau < 1
  }

  // lo <= v* <= hi; c_lo masses are >= lo, c_hi are > hi, and above = F(hi + 1).
  // find_blocks: the masses below v add up to less than m v, so F(v) >= target
  // for every v <= slack / m.
  uint32_t lo = COUNT ? 0u : (uint32_t)((float)slack * 0.999f / (float)m);
  lo = COUNT || lo > 1u ? lo : 1u;
  if constexpr (LEAST) {  // F is the whole total up to the least mass
    least = ~wave_max_u32(~least);
    lo = lo > least ? lo : least;
  }
  uint32_t hi = wave_max_u32(top);
  uint32_t c_lo = (uint32_t)m, c_hi = 0;
  uint64_t above = 0;
  while (NPL > 1 && c_lo - c_hi > 64u && lo < hi) {
    uint32_t mid;
    if (hi >> 1 > lo) {
      mid = (uint32_t)__builtin_amdgcn_readfirstlane(
          (int)(uint32_t)__builtin_amdgcn_sqrtf((float)(lo > 1u ? lo : 1u) * (float)hi));
      mid = mid > lo ? (mid < hi ? mid : hi) : lo + 1u;
    } else {
      mid = lo + ((hi - lo - 1u) >> 1) + 1u;
    }
    uint64_t f = 0;
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const bool in = u[i] >= mid;  // mid >= 1: never a padding slot
      n += (uint32_t)__popcll(__ballot(in));
      if constexpr (!COUNT) f += in ? u[i] : 0u;
    }
    f = COUNT ? (uint64_t)n : wave_sum_u64(f) + ones;
    if (f >= target) {
      lo = mid;
      c_lo = n;
    } else {
      hi = mid - 1u;
      c_hi = n;
      above = f;
    }
  }

  uint32_t vstar = lo, ties = 0;
  uint64_t reach = 0;  // F(v*)
  if (c_lo - c_hi <= 64u) {
    // the masses in [lo, hi], one per lane; `held` marks the lanes
    uint32_t c;
    uint64_t held;
    if constexpr (NPL == 1) {
      c = u[0];
      held = __ballot(lane < m && c >= lo);
    } else {
      uint32_t pos = 0;
#pragma unroll
      for (int i = 0; i < NPL; ++i) {
        const bool in = lane + 64 * i < m && u[i] >= lo && u[i] <= hi;
        const uint64_t msk = __ballot(in);
        if (in) stage[pos + rank_in(msk)] = u[i];
        pos += (uint32_t)__popcll(msk);
      }
      __builtin_amdgcn_wave_barrier();
      c = lane < (int)pos ? stage[lane] : 0u;
      held = pos >= 64u ? ~0ull : (1ull << pos) - 1ull;
    }
    // each lane: what the masses not below its own add up to
    uint64_t f = above + (!COUNT && hi == 0xFFFFFFFFu ? ones : 0u);
    for (uint64_t left = held; left != 0; left &= left - 1ull) {
      const uint32_t x = __builtin_amdgcn_readlane(c, (int)__builtin_ctzll(left));
      f += x >= c ? (COUNT ? 1u : x) : 0u;
    }
    const bool ok = (held >> lane & 1ull) && f >= target;
    vstar = wave_max_u32(ok ? c : 0u);
    const uint64_t tmask = __ballot(ok && c == vstar);
    ties = (uint32_t)__popcll(tmask);
    const int first = (int)__builtin_ctzll(tmask);
    reach = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)f, first) |
            (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(f >> 32), first) << 32;
  } else {  // lo == hi; c_lo may still be the initial bound
#pragma unroll
    for (int i = 0; i < NPL; ++i)
      ties += (uint32_t)__popcll(__ballot(u[i] == vstar && lane + 64 * i < m));
    reach = above + (COUNT ? (uint64_t)ties : (uint64_t)ties * mass(vstar));
  }
  // the ties that bring F(v* + 1) = reach - ties v* to the target
  uint32_t ties_needed = ties;
  if (ties > 1) {
    const uint64_t w = mass(vstar), base = reach - (COUNT ? (uint64_t)ties : ties * w);
    ties_needed = (uint32_t)(COUNT ? target - base : (target - base + w - 1) / w);
  }

  uint32_t written = 0, ties_seen = 0;
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    const int j = lane + 64 * i;
    bool sel = u[i] >= vstar && j < m;
    if (ties_needed != ties) {  // uniform
      const bool tie = sel && u[i] == vstar;
      const uint64_t tmask = __ballot(tie);
      if (tie && ties_seen + rank_in(tmask) >= ties_needed) sel = false;
      ties_seen += (uint32_t)__popcll(tmask);
    }
    const uint64_t smask = __ballot(sel);
    if (sel) out[written + rank_in(smask)] = j;
    written += (uint32_t)__popcll(smask);
  }
  if (lane == 0) *cnt_out = (int32_t)written;
}

template <int NPL, bool COUNT>
__device__ __forceinline__ void select_row_sized(const float* s, int m, float tau, int k,
                                                 int lane, int32_t* out, int32_t* cnt_out,
                                                 uint32_t* stage) {
  const int nact = (m + 63) >> 6;
  // Rows of nearly equal masses (queries that attend evenly) need up to 25
  // steps from a bracket ten times wide. Where 128 candidates are the most, the
  // least mass is free (128 blocks, 32 heads, masses within 1e-6 of each other
  // 15.6 -> 9.4 us, others 9.0-9.4 us as before); longer rows would pay 2-4 %
  // for it with every other distribution.
  constexpr bool kLeast = NPL == 2;
  if (NPL <= 1 || nact <= 1) select_row<1, COUNT>(s, m, tau, k, lane, out, cnt_out, stage);
  else if (NPL <= 2 || nact <= 2) select_row<(NPL < 2 ? NPL : 2), COUNT, kLeast>(s, m, tau, k, lane, out, cnt_out, stage);
  else if (NPL <= 4 || nact <= 4) select_row<(NPL < 4 ? NPL : 4), COUNT>(s, m, tau, k, lane, out, cnt_out, stage);
  else if (NPL <= 8 || nact <= 8) select_row<(NPL < 8 ? NPL : 8), COUNT>(s, m, tau, k, lane, out, cnt_out, stage);
  else if (NPL <= 16 || nact <= 16) select_row<(NPL < 16 ? NPL : 16), COUNT>(s, m, tau, k, lane, out, cnt_out, stage);
  else select_row<NPL, COUNT>(s, m, tau, k, lane, out, cnt_out, stage);
}

}  // namespace xattn

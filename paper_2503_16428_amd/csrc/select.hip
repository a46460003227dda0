// Step 2: the selection kernel and its launches; the search of one row is in
// select_rows.h.
#include "select_rows.h"

using namespace xattn;

namespace {

// One wave64 per (head, query block) row. NPL = slots per lane for the
// longest row (64 NPL >= NB); a causal row with m = b + 1 candidates runs the
// smallest power-of-two slot count that holds them. Per-head parameters are
// indexed by the row's head modulo hq (the same for every batch element).
template <int NPL, bool CAUSAL>
__global__ __launch_bounds__(256) void select_kernel(const float* __restrict__ scores,
                                                     int n_rows, int NB, SelectParams p,
                                                     int32_t* __restrict__ idx,
                                                     int32_t* __restrict__ cnt) {
  __shared__ uint32_t stage_all[4][64];  // per wave: the values left for the search's end
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;  // uniform per wave
  const int b = row % NB;
  const int hp = p.uniform ? 0 : (row / NB) % p.hq;
  const int m = CAUSAL ? b + 1 : NB;
  const float* s = scores + (size_t)row * NB;
  int32_t* out = idx + (size_t)row * NB;

  int k = m;  // blocks a fixed-size mode keeps
  if (p.mode == kSelectTopK) {
    k = p.k[hp];
  } else if (p.mode == kSelectRatio) {
    const double want = floor((double)p.v[hp] * (double)m + 0.5);
    k = want < 1.0 ? 1 : (want > (double)m ? m : (int)want);
  }
  k = k < 1 ? 1 : k;
  const bool all = p.mode == kSelectThreshold ? p.v[hp] >= 1.f : k >= m;
  if (all) {
    for (int j = lane; j < m; j += 64) out[j] = j;
    if (lane == 0) cnt[row] = m;
    return;
  }
  uint32_t* stage = stage_all[threadIdx.x >> 6];
  if (p.mode == kSelectThreshold)
    select_row_sized<NPL, false>(s, m, p.v[hp], 0, lane, out, cnt + row, stage);
  else
    select_row_sized<NPL, true>(s, m, 0.f, k, lane, out, cnt + row, stage);
}

template <int NPL>
hipError_t launch_npl(const float* scores, const XattnShape& s, const SelectParams& p,
                      int32_t* idx, int32_t* cnt, hipStream_t st) {
  const int n_rows = s.HQ() * s.NB();
  const dim3 grid((n_rows + 3) / 4);
  if (s.causal)
    hipLaunchKernelGGL((select_kernel<NPL, true>), grid, dim3(256), 0, st, scores, n_rows,
                       s.NB(), p, idx, cnt);
  else
    hipLaunchKernelGGL((select_kernel<NPL, false>), grid, dim3(256), 0, st, scores, n_rows,
                       s.NB(), p, idx, cnt);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const float* scores, const XattnShape& s, const SelectParams& p,
                         int32_t* idx, int32_t* cnt, hipStream_t st) {
  const int NB = s.NB();
  if (NB <= 64) return launch_npl<1>(scores, s, p, idx, cnt, st);
  if (NB <= 128) return launch_npl<2>(scores, s, p, idx, cnt, st);
  if (NB <= 256) return launch_npl<4>(scores, s, p, idx, cnt, st);
  if (NB <= 512) return launch_npl<8>(scores, s, p, idx, cnt, st);
  if (NB <= 1024) return launch_npl<16>(scores, s, p, idx, cnt, st);
  if (NB <= 2048) return launch_npl<32>(scores, s, p, idx, cnt, st);
  return hipErrorInvalidValue;
}

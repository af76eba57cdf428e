// gather_tile.h -- device pieces shared by the gathers (gather.hip,
// gather_split.hip), the fp32 model's one-kernel path (net_f32.hip), the
// network over row tiles (net_rows.hip) and the literal SE layer
// (se_literal.hip).
#pragma once

#include "cold_internal.h"

namespace cold {

// last q with req_off[q] <= r, clamped to [0, Q-1]
__device__ __forceinline__ int64_t request_of_row(const int32_t *req_off, int64_t Q, int64_t r) {
  int64_t lo = 0, hi = Q;  // invariant: answer in [lo, hi)
  while (hi - lo > 1) {
    int64_t mid = (lo + hi) >> 1;
    if ((int64_t)req_off[mid] <= r) lo = mid; else hi = mid;
  }
  return lo;
}

// Eq. 3: identity on [-1, 1], sign(x) (1 + ln|x|) outside, branch-free.  The
// natural log comes from the hardware log2 (relative error near 2^-22),
// far below the half-precision rounding that follows it.
__device__ __forceinline__ float linear_log(float x) {
  const float ax = fabsf(x);
  const float l = __logf(ax) + 1.0f;   // used only when |x| > 1
  return ax > 1.0f ? copysignf(l, x) : x;
}

// Eq. 3 on a lane's N values. It leaves |x| <= 1 as it is, so the logarithms
// (a quarter-rate instruction and six more each) run only where a lane of
// the wave holds a larger value: a pooled sequence, hardly ever an embedding.
template <int N>
__device__ __forceinline__ void linear_log_all(float (&v)[N]) {
  float m = 0.0f;
#pragma unroll
  for (int e = 0; e < N; ++e) m = fmaxf(m, fabsf(v[e]));
  if (__any(m > 1.0f)) {
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = linear_log(v[e]);
  }
}

// shape limits of the register-resident gathers
constexpr int kFullMaxM = 64;
constexpr int kFullMaxH = 16;
constexpr int kFullTileM = 48;   // the one-wave-per-tile form up to this many groups

}  // namespace cold

// Multi-Krum's selection by one wave, shared by the short inputs' combined
// kernel (select.hip) and the guess before a long distance pass
// (ring_direct.hip).
#pragma once

#include "device_common.h"
#include "dist_layout.h"

namespace garfield {

// Multi-Krum's selection from the N x N distances (entry sums esum, direct
// layout), by the 64 lanes of one wave without LDS traffic or barriers: lane
// i < N sorts its row's N-1 distances, adds the k = N-f-2 smallest as the
// butterfly of krum_flags adds them (a balanced tree in ascending order, the
// other slots 0: the same bits), and ranks its (score, i) against every
// lane's. Returns the lane-uniform mask of the m selected rows.
template <int N>
__device__ __forceinline__ uint64_t krum_mask_wave(const double* esum, int f, int m) {
  constexpr int M = N - 1;
  const int i = threadIdx.x & 63;
  const int k = N - f - 2;
  double score = 0.0;
  if (i < N) {
    double r[M];
#pragma unroll
    for (int q = 0; q < M; ++q) {
      const int j = q < i ? q : q + 1;
      r[q] = esum[direct_entry(N, i < j ? i : j, i < j ? j : i)];
    }
#pragma unroll
    for (int a = 0; a < M; ++a)  // bubble network: ascending
#pragma unroll
      for (int b = 0; b + 1 < M - a; ++b) {
        const double lo = __builtin_fmin(r[b], r[b + 1]);
        r[b + 1] = __builtin_fmax(r[b], r[b + 1]);
        r[b] = lo;
      }
    constexpr int T = M <= 16 ? 16 : 32;
    double t[T];
#pragma unroll
    for (int q = 0; q < T; ++q) t[q] = (q < M && q < k) ? r[q < M ? q : 0] : 0.0;
#pragma unroll
    for (int h = 1; h < T; h <<= 1)
#pragma unroll
      for (int q = 0; q < T; q += 2 * h) t[q] = t[q] + t[q + h];
    score = t[0];
  }
  const int64_t bits = __double_as_longlong(score);
  const int lo = static_cast<int>(bits), hi = static_cast<int>(bits >> 32);
  int rank = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const uint64_t sj_bits =
        (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(hi, j))) << 32) |
        static_cast<uint32_t>(__builtin_amdgcn_readlane(lo, j));
    const double sj = __longlong_as_double(static_cast<int64_t>(sj_bits));
    rank += (sj < score) | ((sj == score) & (j < i));
  }
  return __ballot(i < N && rank < m);
}

}  // namespace garfield

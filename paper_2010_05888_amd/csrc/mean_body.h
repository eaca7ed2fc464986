// The mean of k rows per coordinate, shared by the kernels over one matrix
// (aggregate.hip, ring_direct.hip), over a table of segments (segtable.hip) and
// over many nodes (contract.hip), with the row rules the other gathers use too.
#pragma once

#include "device_common.h"
#include "internal.h"
#include "rows.h"

namespace garfield {

// The rows a body reads, as a type, so that its loop over the rows has no
// branch: AllRows reads rows 0 .. k-1, ListedRows the listed ones. Kernels
// given an optional list come in both forms and the host picks one: a choice
// made per row made each row's load wait for the scalar load of its own
// index, where branch-free indices are fetched together ahead of the loads.
struct AllRows {
  __device__ __forceinline__ int64_t operator()(int t) const { return t; }
};

// An index outside [0, n) breaks a precondition; it reads row n - 1 rather
// than memory outside the input (one unsigned minimum, and the row offset is
// then an unsigned 32 x 64-bit product: few scalar instructions per row).
struct ListedRows {
  const int32_t* list;
  int n;
  __device__ __forceinline__ int64_t operator()(int t) const {
    const uint32_t r = static_cast<uint32_t>(list[t]);
    const uint32_t last = static_cast<uint32_t>(n - 1);
    return static_cast<int64_t>(r < last ? r : last);
  }
};

// Row t of an optional list (rows 0 .. k-1 without one), by ListedRows' rule;
// for code outside the gathers' loops (staging, masks).
__device__ __forceinline__ int64_t row_of(const int32_t* __restrict__ rows, int t, int n) {
  return rows ? ListedRows{rows, n}(t) : static_cast<int64_t>(t);
}

// sum / count, correctly rounded, as the division gives it (count a whole
// number of at most kNmax, inv = 1 / count rounded): with inv within half an
// ulp of 1 / count and q = sum * inv, one residual step is exact for every sum
// whose quotient is normal (Markstein's theorem), and the fixup passes
// infinities and NaN through. Four instructions where the general division
// takes about twelve.
__device__ __forceinline__ double mean_of(double sum, double count, double inv) {
  const double q = sum * inv;
  const double r = __builtin_fma(-q, count, sum);
  return __builtin_amdgcn_div_fixup(__builtin_fma(r, inv, q), count, sum);
}

template <int W>
__device__ __forceinline__ void store_out(float* __restrict__ out, int64_t c, int64_t d,
                                          bool full, const float* o) {
  if (full) {
    store_w<W>(out + c, o);
  } else {
    for (int e = 0; e < W && c + e < d; ++e) out[c + e] = o[e];
  }
}

// ---------------------------------------------------------------------------
// Mean of k rows: fp64 sum of the rows in the order listed, eight loads in
// flight at a time, one rounding at the end.
template <int W, bool FULL, bool NT, class Src, class L>
__device__ __forceinline__ void sum_rows_at(const Src& src, int64_t d, const L& rows, int k,
                                            int64_t c, double* acc) {
  int t = 0;
  for (; t + 8 <= k; t += 8) {
    float v[8][W];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float* p = src.row(rows(t + u)) + c;
      if constexpr (FULL) load_w<W, NT>(p, v[u]); else load_w_tail<W>(p, d - c, v[u]);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < W; ++e) acc[e] += static_cast<double>(v[u][e]);
  }
  for (; t < k; ++t) {
    float v[W];
    const float* p = src.row(rows(t)) + c;
    if constexpr (FULL) load_w<W, NT>(p, v); else load_w_tail<W>(p, d - c, v);
#pragma unroll
    for (int e = 0; e < W; ++e) acc[e] += static_cast<double>(v[e]);
  }
}

template <int W, bool NT = true, class Src, class L>
__device__ __forceinline__ void mean_at(const Src& src, int64_t d, const L& rows, int k,
                                        int64_t c, float* __restrict__ out) {
  double acc[W];
#pragma unroll
  for (int e = 0; e < W; ++e) acc[e] = 0.0;
  const bool full = c + W <= d;
  if (full) sum_rows_at<W, true, NT>(src, d, rows, k, c, acc);
  else sum_rows_at<W, false, NT>(src, d, rows, k, c, acc);
  const double count = static_cast<double>(k);
  float o[W];
#pragma unroll
  for (int e = 0; e < W; ++e) o[e] = static_cast<float>(acc[e] / count);
  store_out<W>(out, c, d, full, o);
}

// The mean of k distinct rows (sel, ascending; `chosen` their mask, n rows in
// all) at the W coordinates c .. c+W-1 from the column sums: where all of them
// are exact (not NaN) the rows not chosen are subtracted in ascending order,
// two rows' loads in flight; otherwise the rows of sel are summed as mean_at
// sums them. Either way the fp64 value is the exact sum mean_at forms (sums of
// these values are exact where the column sum is), rounded once.
template <int W, class Src>
__device__ __forceinline__ void complement_at(const Src& src, int n, int64_t d,
                                              const int32_t* __restrict__ sel, int k,
                                              uint64_t chosen, const double* __restrict__ colsum,
                                              int64_t c, float* __restrict__ out) {
  const bool full = c + W <= d;
  double acc[W];
  bool loaded = false;
  if constexpr (W >= 2) {
    if (full) {  // ordinary 16-byte loads: a line's halves meet in L2
#pragma unroll
      for (int e = 0; e < W; e += 2) {
        const d2 t = *reinterpret_cast<const d2*>(colsum + c + e);
        acc[e] = t.x;
        acc[e + 1] = t.y;
      }
      loaded = true;
    }
  }
  if (!loaded) {
#pragma unroll
    for (int e = 0; e < W; ++e) acc[e] = (c + e < d) ? colsum[c + e] : 0.0;
  }
  bool exact = true;
#pragma unroll
  for (int e = 0; e < W; ++e) exact = exact && !__builtin_isnan(acc[e]);
  if (exact) {
    uint64_t rest = ~chosen & (n == 64 ? ~uint64_t{0} : (uint64_t{1} << n) - 1);  // uniform
    while (rest) {
      const int r0 = __builtin_ctzll(rest);
      rest &= rest - 1;
      const bool two = rest != 0;
      const int r1 = two ? __builtin_ctzll(rest) : r0;
      rest &= rest - 1;
      float v[2][W];
      const float* p0 = src.row(r0) + c;
      const float* p1 = src.row(r1) + c;
      if (full) {
        load_w<W>(p0, v[0]);
        load_w<W>(p1, v[1]);
      } else {
        load_w_tail<W>(p0, d - c, v[0]);
        load_w_tail<W>(p1, d - c, v[1]);
      }
#pragma unroll
      for (int e = 0; e < W; ++e) acc[e] -= static_cast<double>(v[0][e]);
      if (two) {
#pragma unroll
        for (int e = 0; e < W; ++e) acc[e] -= static_cast<double>(v[1][e]);
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < W; ++e) acc[e] = 0.0;
    if (full) sum_rows_at<W, true, true>(src, d, ListedRows{sel, n}, k, c, acc);
    else sum_rows_at<W, false, true>(src, d, ListedRows{sel, n}, k, c, acc);
  }
  const double count = static_cast<double>(k);
  float o[W];
#pragma unroll
  for (int e = 0; e < W; ++e) o[e] = static_cast<float>(acc[e] / count);
  store_out<W>(out, c, d, full, o);
}

// The mask of the k rows listed in sel (the same in every lane).
__device__ __forceinline__ uint64_t rows_mask(const int32_t* __restrict__ sel, int k, int n) {
  uint64_t mask = 0;
  for (int t = 0; t < k; ++t) mask |= uint64_t{1} << row_of(sel, t, n);
  return mask;
}

}  // namespace garfield

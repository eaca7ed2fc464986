// Per-coordinate bodies of the streaming aggregation kernels, shared by the
// kernels over one row-major matrix (aggregate.hip) and the kernels over a
// table of segments (segtable.hip). Each body handles W consecutive
// coordinates c .. c+W-1 of a segment of length d and writes them to out + c;
// the rows come from a source (rows.h) and a row rule (AllRows, ListedRows)
// says which of them are used. NT: nontemporal loads (rows read once); kernels whose
// workgroups share rows read them with ordinary loads, which stay in L2.
#pragma once

#include "device_common.h"
#include "internal.h"
#include "mean_body.h"
#include "rows.h"

namespace garfield {

#include "networks.inc"

// ---------------------------------------------------------------------------
// Coordinate-wise median of K rows: all K loads back to back, then the
// selection network per coordinate.
template <int K, int W, bool NT = true, class Src, class L>
__device__ __forceinline__ void median_at(const Src& src, int64_t d, const L& rows, int64_t c,
                                          float* __restrict__ out) {
  using Net = MedianNet<K>;
  float v[K][W];
  const bool full = c + W <= d;
  if (full) {
#pragma unroll
    for (int t = 0; t < K; ++t) load_w<W, NT>(src.row(rows(t)) + c, v[t]);
  } else {
#pragma unroll
    for (int t = 0; t < K; ++t) load_w_tail<W>(src.row(rows(t)) + c, d - c, v[t]);
  }
  float o[W];
#pragma unroll
  for (int e = 0; e < W; ++e) {
    float a[K];
#pragma unroll
    for (int t = 0; t < K; ++t) a[t] = v[t][e];
    Net::run(a);
    if constexpr (K % 2 == 1) {
      o[e] = a[Net::LO];
    } else {  // mean of the two middle values, exact in fp64, rounded once
      o[e] = static_cast<float>((static_cast<double>(a[Net::LO]) +
                                 static_cast<double>(a[Net::HI])) * 0.5);
    }
  }
  store_out<W>(out, c, d, full, o);
}

// ---------------------------------------------------------------------------
// Bulyan with beta = 3 (theta = 2f + 3, the smallest n for f, so T is odd):
// only the ranks c-2 .. c+2 around the median s[c] can be taken, so a band
// network (BandNet) leaves them in registers and the rule below -- the same
// comparisons and the same fp64 sum as bulyan_at's general path -- runs on
// compile-time registers, without the LDS column.
template <int T>
__device__ __forceinline__ float bulyan3_of_band(const float* a) {
  using B = BandNet<T>;
  constexpr int c = (T - 1) / 2;  // n_left = n_right = c
  const double med = static_cast<double>(a[B::reg(c)]);
  auto take = [&](float lv, float rv) {  // L before R in the merge by (|v - med|, v)
    const double dl = med - static_cast<double>(lv);
    const double dr = static_cast<double>(rv) - med;
    return (dl < dr) || (dl == dr && lv < rv);
  };
  double sum = 0.0;
  if constexpr (T == 3) {  // the whole set
    sum += static_cast<double>(a[B::reg(0)]);
    sum += static_cast<double>(a[B::reg(1)]);
    sum += static_cast<double>(a[B::reg(2)]);
  } else {
    // L_1 = s[c-1] against R_2 = s[c+2], then L_2 = s[c-2] against R_1 = s[c+1]
    int a_taken = 0;
    if (take(a[B::reg(c - 1)], a[B::reg(c + 2)])) {
      a_taken = 1;
      if (take(a[B::reg(c - 2)], a[B::reg(c + 1)])) a_taken = 2;
    }
    const float x0 = a_taken == 0 ? a[B::reg(c)] : (a_taken == 1 ? a[B::reg(c - 1)] : a[B::reg(c - 2)]);
    const float x1 = a_taken == 0 ? a[B::reg(c + 1)] : (a_taken == 1 ? a[B::reg(c)] : a[B::reg(c - 1)]);
    const float x2 = a_taken == 0 ? a[B::reg(c + 2)] : (a_taken == 1 ? a[B::reg(c + 1)] : a[B::reg(c)]);
    sum += static_cast<double>(x0);
    sum += static_cast<double>(x1);
    sum += static_cast<double>(x2);
  }
  return static_cast<float>(sum / 3.0);
}

// ---------------------------------------------------------------------------
// Bulyan aggregation for theta = T selected rows, beta = T - 2f closest.
//
// With s[0..T-1] sorted: odd T has the median s[c], c = (T-1)/2, always kept,
// and K = beta-1 more to take; even T has med = (s[c-1]+s[c])/2, c = T/2, and
// K = beta to take. Left candidates L_a = s[c-a] (a = 1, 2, ...) and right
// candidates R_b (s[c+b] for odd T, s[c-1+b] for even T) are each ordered by
// increasing key, so the K taken are the first K of their merge: L_a is taken
// iff key(L_a) < key(R_{K+1-a}) (a missing R counts as +inf). The number of
// left values taken is the count of such a. `col` is this thread's column of
// a T x kBlock LDS array (col[r * kBlock]).
template <int T, int W, bool NT = true, class Src, class L>
__device__ __forceinline__ void bulyan_at(const Src& src, int64_t d, const L& sel, int beta,
                                          int64_t cc, float* col, float* __restrict__ out) {
  using Net = SortNet<T>;
  constexpr bool kOdd = (T % 2) == 1;
  constexpr int c = kOdd ? (T - 1) / 2 : T / 2;
  constexpr int n_left = c;                          // L_a exists for a <= n_left
  constexpr int n_right = kOdd ? T - 1 - c : T - c;  // R_b exists for b <= n_right
  const int K = kOdd ? beta - 1 : beta;
  float v[T][W];
  const bool full = cc + W <= d;
  if (full) {
#pragma unroll
    for (int t = 0; t < T; ++t) load_w<W, NT>(src.row(sel(t)) + cc, v[t]);
  } else {
#pragma unroll
    for (int t = 0; t < T; ++t) load_w_tail<W>(src.row(sel(t)) + cc, d - cc, v[t]);
  }
  float o[W];
  if constexpr (kOdd && T >= 3) {
    if (beta == 3) {  // uniform: the band network and registers only
#pragma unroll
      for (int e = 0; e < W; ++e) {
        float a[T];
#pragma unroll
        for (int t = 0; t < T; ++t) a[t] = v[t][e];
        BandNet<T>::run(a);
        o[e] = bulyan3_of_band<T>(a);
      }
      store_out<W>(out, cc, d, full, o);
      return;
    }
  }
#pragma unroll
  for (int e = 0; e < W; ++e) {
    float a[T];
#pragma unroll
    for (int t = 0; t < T; ++t) a[t] = v[t][e];
    Net::run(a);
#pragma unroll
    for (int r = 0; r < T; ++r) col[r * kBlock] = a[Net::reg(r)];
    const double med = kOdd ? static_cast<double>(col[c * kBlock])
                            : (static_cast<double>(col[(c - 1) * kBlock]) +
                               static_cast<double>(col[c * kBlock])) * 0.5;
    int a_taken = 0;
    for (int i = 1; i <= K; ++i) {
      if (i > n_left) break;
      const int b = K + 1 - i;
      bool take = true;
      if (b <= n_right) {
        const float lv = col[(c - i) * kBlock];
        const float rv = col[(kOdd ? c + b : c - 1 + b) * kBlock];
        const double dl = med - static_cast<double>(lv);
        const double dr = static_cast<double>(rv) - med;
        take = (dl < dr) || (dl == dr && lv < rv);
      }
      if (!take) break;
      a_taken = i;
    }
    const int lo = c - a_taken;
    const int hi = lo + beta - 1;  // inclusive
    double sum = 0.0;
    for (int r = lo; r <= hi; ++r) sum += static_cast<double>(col[r * kBlock]);
    o[e] = static_cast<float>(sum / static_cast<double>(beta));
  }
  store_out<W>(out, cc, d, full, o);
}

}  // namespace garfield

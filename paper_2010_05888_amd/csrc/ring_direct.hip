// The direct distance engine for long inputs: rows streamed through an LDS
// ring (ring.h) by one persistent workgroup per CU, and with it the mean of a
// selection guessed beforehand, so that a rule whose selection is clear reads
// its input once.
//
// Why a ring. The register form (direct_body.h) keeps its loads in flight in
// the registers its accumulators need too, so from 13 rows on it had to load 8
// bytes a lane, and at any n its loads in flight fell with its occupancy. Here
// the loads go to LDS, 80 to 120 KB of them per CU at any n, and the registers
// hold accumulators only. Up to 12 rows the pass is bound by HBM: n = 11 at
// 25.6 M coordinates 169 us, 6.65 TB/s (register form 190 us, 5.92), where a
// plain read of one contiguous buffer reaches 6.9. From 16 rows on it is bound
// by the vector unit, two instructions per pair and coordinate: n = 19 349 us,
// its VALU busy 90 % of the time at 2.0 GHz, and 330 to 500 as the clock goes
// (register form 402 us). Tried and slower: every group reading all rows from
// LDS (n = 17: 344 against 327 us), and one barrier per stage without the next
// stage's LDS reads ahead of it (n = 14: 256 against 244 us).
//
// The mean it writes: 25.6 M coordinates, n = 10, m = 7, MDA's call 322 -> 225
// us (the distance pass 174 -> 190 us, the mean's own pass of 134 us gone);
// n = 11, m = 9 at 11.2 M, Multi-Krum's 150 -> 110 us.

#include <utility>

#include "device_common.h"
#include "direct_body.h"
#include "dist_layout.h"
#include "internal.h"
#include "krum_mask.h"
#include "mean_body.h"
#include "ring.h"
#include "timing.h"

namespace garfield {

namespace {

// The pairs are split over GROUPS groups of waves that read the rows from LDS,
// so that a lane's accumulators (fp32, and the fp64 they are added into every
// 16 coordinates) fit two waves per SIMD. Every group gives its lanes the same
// coordinates and every pair is summed by the same tree, so identical rows
// give bit-identical rows of D wherever they sit.
//
// Four groups split the rows into A = [0, a) and B = [a, n): the pairs inside
// A, those inside B, and the pairs of A with the first k rows of B and with
// the rest. No group reads all rows, and waves w and w + 4, which share a SIMD,
// hold groups 0 and 2 or 1 and 3: a and k are the split whose two sums are
// nearest (then the one that reads the fewest rows).
struct PairSplit {
  int a, k;
};
constexpr PairSplit pair_split(int n) {
  PairSplit best{1, 0};
  int cost = 1 << 30;
  for (int a = 2; a <= n - 2; ++a)
    for (int k = 1; k <= n - a - 1; ++k) {
      const int g0 = a * (a - 1) / 2, g1 = (n - a) * (n - a - 1) / 2;
      const int g2 = a * k, g3 = a * (n - a - k);
      const int s0 = g0 + g2, s1 = g1 + g3;
      int most = g0 > g1 ? g0 : g1;
      most = most > g2 ? most : g2;
      most = most > g3 ? most : g3;
      if (most > 52) continue;  // accumulators per lane
      const int c = (s0 > s1 ? s0 : s1) * 1000 + n + n - a + a + k;
      if (c < cost) {
        cost = c;
        best = PairSplit{a, k};
      }
    }
  return best;
}

template <int N>
struct RingDirect {
  static constexpr int P = N * (N - 1) / 2;
  static constexpr int GROUPS = N <= 10 ? 1 : (N <= 13 ? 2 : 4);
  static constexpr int LANES = kRingThreads / GROUPS;
  static constexpr int COORDS = RingShape<N>::STAGE / LANES;  // per lane and stage
  static constexpr int PASSES = COORDS / 2;                   // of 8-byte LDS reads
  static constexpr int FLUSH = kDirectLaneCoords / COORDS;    // stages per fp32 run
  static constexpr PairSplit SPLIT = pair_split(N < 4 ? 4 : N);
  static_assert(PASSES * 2 * LANES == RingShape<N>::STAGE && (PASSES == 1 || PASSES == 2),
                "8-byte reads cover a stage in one or two passes");
  static_assert(FLUSH * COORDS == kDirectLaneCoords && FLUSH % 2 == 0,
                "whole pairs of stages per fp32 run");

  // the group of pair (i < j) and its place there
  static __host__ __device__ constexpr int group(int i, int j) {
    if (GROUPS == 1) return 0;
    if (GROUPS == 2) return direct_entry(N, i, j) >= P / 2;
    if (j < SPLIT.a) return 0;
    if (i >= SPLIT.a) return 1;
    return j < SPLIT.a + SPLIT.k ? 2 : 3;
  }
  static __host__ __device__ constexpr int place(int i, int j) {
    if (GROUPS == 1) return direct_entry(N, i, j);
    if (GROUPS == 2) return direct_entry(N, i, j) - (group(i, j) ? P / 2 : 0);
    switch (group(i, j)) {
      case 0: return direct_entry(SPLIT.a, i, j);
      case 1: return direct_entry(N - SPLIT.a, i - SPLIT.a, j - SPLIT.a);
      case 2: return i * SPLIT.k + j - SPLIT.a;
      default: return i * (N - SPLIT.a - SPLIT.k) + j - SPLIT.a - SPLIT.k;
    }
  }
  // the pairs of every group by place, their number, and which rows they take
  struct Lists {
    int i[GROUPS][64], j[GROUPS][64], count[GROUPS];
    bool reads[GROUPS][N];
  };
  static constexpr Lists lists() {
    Lists l{};
    for (int i = 0; i < N; ++i)
      for (int j = i + 1; j < N; ++j) {
        const int g = group(i, j), q = place(i, j);
        l.i[g][q] = i;
        l.j[g][q] = j;
        ++l.count[g];
        l.reads[g][i] = l.reads[g][j] = true;
      }
    return l;
  }
  static constexpr Lists L = lists();
  static constexpr int maxcount() {
    int m = 0;
    for (int g = 0; g < GROUPS; ++g) m = L.count[g] > m ? L.count[g] : m;
    return m;
  }
};

// The values of group GRP's rows (ALL: of every row) at this lane's two
// coordinates of pass q.
template <int N, int GRP, bool ALL>
__device__ __forceinline__ void ring_read(const float* __restrict__ slot, int q, int tl, f2* v) {
  using S = RingDirect<N>;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (ALL || S::L.reads[GRP][i])
      v[i] = *reinterpret_cast<const f2*>(slot + i * RingShape<N>::STAGE + 2 * (q * S::LANES + tl));
}

// acc[place] += (x_i - x_j)^2 over them, for the pairs of group GRP; FIRST:
// the first coordinates of an fp32 run (acc is not read).
template <int N, int GRP, bool FIRST, int... Q>
__device__ __forceinline__ void ring_add(const f2* v, float* acc,
                                         std::integer_sequence<int, Q...>) {
  using S = RingDirect<N>;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    auto pair = [&](auto q) {
      constexpr int i = S::L.i[GRP][decltype(q)::value], j = S::L.j[GRP][decltype(q)::value];
      const float t = v[i][e] - v[j][e];
      if (FIRST && e == 0) acc[decltype(q)::value] = t * t;
      else acc[decltype(q)::value] = __builtin_fmaf(t, t, acc[decltype(q)::value]);
    };
    (pair(std::integral_constant<int, Q>{}), ...);
  }
}

// What the pass writes per coordinate beside the distances.
struct RingOut {
  const uint64_t* guess;
  double* colsum;
  float* out;
  int m;
};
enum RingWrites { kNothing = 0, kMean = 1, kColsum = 2 };

// Whether there is a guess and every run's agrees; *mask = it.
__device__ __forceinline__ bool guess_agrees(const uint64_t* __restrict__ guess, uint64_t* mask) {
  if (!guess) return false;
  const uint64_t g0 = guess[0];
  bool same = true;
#pragma unroll
  for (int r = 1; r < kGuessRuns; ++r) same = same && guess[r] == g0;
  *mask = g0;
  return same;
}

// The mean of the rows of `mask` (kMean) or the column sums (kColsum) at the
// two coordinates c, c + 1 whose values v holds; those at or beyond d are left
// out unless FULL. One vector store where FULL.
template <int N, int WRITES, bool FULL>
__device__ __forceinline__ void ring_write(const RingOut& o, uint64_t mask, const f2* v, int64_t c,
                                           int64_t d) {
  if constexpr (WRITES == kMean) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if ((mask >> i) & 1) {  // uniform
        s0 += static_cast<double>(v[i].x);
        s1 += static_cast<double>(v[i].y);
      }
    }
    const double count = static_cast<double>(o.m), inv = 1.0 / count;
    const float r[2] = {static_cast<float>(mean_of(s0, count, inv)),
                        static_cast<float>(mean_of(s1, count, inv))};
    if constexpr (FULL) {
      store_w<2>(o.out + c, r);
    } else {
      if (c < d) o.out[c] = r[0];
      if (c + 1 < d) o.out[c + 1] = r[1];
    }
  } else if constexpr (WRITES == kColsum) {
    ColSum a, b;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      a.add(v[i].x);
      b.add(v[i].y);
    }
    // ordinary (L2-allocating) stores, as the register form's
    if constexpr (FULL) {
      d2 t;
      t.x = a.value();
      t.y = b.value();
      *reinterpret_cast<d2*>(o.colsum + c) = t;
    } else {
      if (c < d) o.colsum[c] = a.value();
      if (c + 1 < d) o.colsum[c + 1] = b.value();
    }
  }
}

// Group GRP's share of the pass. The groups all hold every coordinate, and the
// part of a stage that a wave's lanes hold is written (WRITES) by the wave of one
// group: with two groups waves 0, 1, 6 and 7, one on each SIMD; with four waves 0
// and 5, on two of the four SIMDs.
template <int N, int GRP, int WRITES>
__device__ __forceinline__ void ring_pass(const float* __restrict__ x, int64_t d, float* lds,
                                          const RingOut& o, uint64_t mask, float* acc,
                                          double* sum) {
  using R = RingShape<N>;
  using S = RingDirect<N>;
  constexpr int M = S::L.count[GRP];
  constexpr bool ALL = WRITES != kNothing;
  // 18 rows with the mean leave no register for the lane's number: the compiler
  // kept it in memory, and reading it back there waited for every load in flight
  // (533 us where this takes 463, 25.6 M coordinates and a right guess).
  constexpr bool FRESH = N == 18 && WRITES == kMean;
  using Pairs = std::make_integer_sequence<int, M>;
  const uint32_t lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tl = threadIdx.x - GRP * S::LANES;
  constexpr int WAVES = kRingWaves / S::GROUPS;  // of a group
  const int gw = wave - GRP * WAVES;
  const bool writes = WRITES != kNothing && gw * S::GROUPS / WAVES == GRP;  // wave-uniform
  const MatrixRows src{x, d};
  const int64_t b = xcd_slot(), G = gridDim.x;
  const int64_t full = d / R::STAGE;
  const int cnt = full > b ? static_cast<int>((full - b + G - 1) / G) : 0;
  const int64_t step = G * R::STAGE;
  int64_t c = b * R::STAGE + 2 * tl;  // this lane's coordinates of the stage being read
  auto flush = [&] {
#pragma unroll
    for (int p = 0; p < M; ++p) sum[p] += static_cast<double>(acc[p]);
  };
  if (cnt > 0) {
    RingLoads<N> loads;
    loads.start(src, b * R::STAGE, wave);
    for (int u = 0; u < R::AHEAD && u < cnt; ++u)
      loads.issue(lds + u * R::SLOT, step, wave, FRESH ? fresh_lane() : lane);
    // Each pass's LDS reads are issued before the arithmetic of the pass
    // before it, the first of the next stage's among them: that stage has
    // landed by this one's barrier.
    f2 v[2][N];
    ring_wait<N, R::AHEAD - 1>(R::AHEAD <= cnt, wave);
    lds_barrier();
    ring_read<N, GRP, ALL>(lds, 0, tl, v[0]);
    int next = 1, fill = R::AHEAD;
    const float* slot = lds;
    auto stage = [&](auto odd, auto first, int i) {
      constexpr int A = decltype(odd)::value, B = 1 - A;
      constexpr bool FIRST = decltype(first)::value;
      // stage i + 1 lands; stage i - 1 is read by every wave
      if (WRITES != kNothing && writes && i >= R::AHEAD)
        ring_wait<N, R::AHEAD - 2, (R::AHEAD - 1) * S::PASSES>(i + R::AHEAD <= cnt, wave);
      else
        ring_wait<N, R::AHEAD - 2>(i + R::AHEAD <= cnt, wave);
      lds_barrier();
      if (i + R::AHEAD < cnt)
        loads.issue(lds + fill * R::SLOT, step, wave, FRESH ? fresh_lane() : lane);
      fill = fill + 1 == R::SLOTS ? 0 : fill + 1;
      const float* after = lds + next * R::SLOT;
      next = next + 1 == R::SLOTS ? 0 : next + 1;
      if constexpr (S::PASSES == 2) {
        ring_read<N, GRP, ALL>(slot, 1, tl, v[1]);
        ring_add<N, GRP, FIRST>(v[0], acc, Pairs{});
        if (writes) ring_write<N, WRITES, true>(o, mask, v[0], c, d);
        if (i + 1 < cnt) ring_read<N, GRP, ALL>(after, 0, tl, v[0]);
        ring_add<N, GRP, false>(v[1], acc, Pairs{});
        if (writes) ring_write<N, WRITES, true>(o, mask, v[1], c + 2 * S::LANES, d);
      } else {
        if (i + 1 < cnt) ring_read<N, GRP, ALL>(after, 0, tl, v[B]);
        ring_add<N, GRP, FIRST>(v[A], acc, Pairs{});
        if (writes) ring_write<N, WRITES, true>(o, mask, v[A], c, d);
      }
      slot = after;
      c += step;
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    for (int i = 0; i < cnt;) {  // one fp32 run of FLUSH stages, or what is left
      const int end = i + S::FLUSH < cnt ? i + S::FLUSH : cnt;
      if constexpr (S::PASSES == 2) {
#pragma unroll
        for (int p = 0; p < M; ++p) acc[p] = 0.0f;
        while (i < end) stage(even, std::false_type{}, i++);
      } else {  // the two stages' values alternate registers
        stage(even, std::true_type{}, i++);
        if (i < end) stage(odd, std::false_type{}, i++);
        while (i + 1 < end) {
          stage(even, std::false_type{}, i++);
          stage(odd, std::false_type{}, i++);
        }
        if (i < end) stage(even, std::false_type{}, i++);
      }
      flush();
    }
  }
  // the partial stage at the end of the rows, staged with guarded loads
  if (d % R::STAGE != 0 && full % G == b) {
    lds_barrier();
    const int64_t c0 = full * R::STAGE;
    for (int idx = threadIdx.x; idx < R::SLOT; idx += kRingThreads) {
      const int64_t cc = c0 + idx % R::STAGE;
      lds[idx] = cc < d ? src.row(idx / R::STAGE)[cc] : 0.0f;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < S::PASSES; ++q) {
      f2 v[N];
      ring_read<N, GRP, ALL>(lds, q, tl, v);
      if (q == 0) ring_add<N, GRP, true>(v, acc, Pairs{});
      else ring_add<N, GRP, false>(v, acc, Pairs{});
      if (writes) ring_write<N, WRITES, false>(o, mask, v, c0 + 2 * (q * S::LANES + tl), d);
    }
    flush();
  }
}

template <int N, int GRP, bool MEAN>
__device__ __forceinline__ void ring_direct(const float* __restrict__ x, int64_t d, float* lds,
                                            double* __restrict__ partial, const RingOut& o) {
  using S = RingDirect<N>;
  constexpr int M = S::L.count[GRP];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float acc[M];
  double sum[M];
#pragma unroll
  for (int p = 0; p < M; ++p) sum[p] = 0.0;
  if constexpr (MEAN) {
    uint64_t mask;
    if (guess_agrees(o.guess, &mask)) {
      ring_pass<N, GRP, kMean>(x, d, lds, o, mask, acc, sum);
    } else if constexpr (N <= kColSumMaxN) {  // no call of more rows takes column sums
      if (o.colsum) ring_pass<N, GRP, kColsum>(x, d, lds, o, 0, acc, sum);
      else ring_pass<N, GRP, kNothing>(x, d, lds, o, 0, acc, sum);
    } else {
      ring_pass<N, GRP, kNothing>(x, d, lds, o, 0, acc, sum);
    }
  } else {
    ring_pass<N, GRP, kNothing>(x, d, lds, o, 0, acc, sum);
  }
  lds_barrier();  // the ring is read; its memory holds the waves' sums now
  double* red = reinterpret_cast<double*>(lds);
  using WS = WaveSums<S::maxcount(), double>;
  double v[WS::P];
#pragma unroll
  for (int p = 0; p < WS::P; ++p) v[p] = p < M ? sum[p < M ? p : 0] : 0.0;
  const double t = WS::run(v, lane);
  if (WS::holds(lane)) red[wave * WS::P + WS::index(lane)] = t;
  lds_barrier();
  constexpr int W = kRingWaves / S::GROUPS;  // waves of a group
  if (static_cast<int>(threadIdx.x) < S::P) {
    int i = 0, j = threadIdx.x;
    while (j >= N - 1 - i) {
      j -= N - 1 - i;
      ++i;
    }
    j += i + 1;
    const double* col = red + S::group(i, j) * W * WS::P + S::place(i, j);
    double a = col[0];
#pragma unroll
    for (int w = 1; w < W; ++w) a += col[w * WS::P];
    partial[static_cast<int64_t>(threadIdx.x) * gridDim.x + blockIdx.x] = a;
  }
}

template <int N, bool MEAN>
__global__ __launch_bounds__(kRingThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_dist_ring(const float* __restrict__ x, int64_t d, double* __restrict__ partial, RingOut o) {
  using S = RingDirect<N>;
  __shared__ __attribute__((aligned(16))) float lds[RingShape<N>::SLOTS * RingShape<N>::SLOT];
  // the group is a compile-time constant per wave, so that its pairs, and
  // with them its registers, are
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / S::LANES);
  if constexpr (S::GROUPS == 1) {
    ring_direct<N, 0, MEAN>(x, d, lds, partial, o);
  } else if constexpr (S::GROUPS == 2) {
    if (grp == 0) ring_direct<N, 0, MEAN>(x, d, lds, partial, o);
    else ring_direct<N, 1, MEAN>(x, d, lds, partial, o);
  } else {
    switch (grp) {
      case 0: ring_direct<N, 0, MEAN>(x, d, lds, partial, o); break;
      case 1: ring_direct<N, 1, MEAN>(x, d, lds, partial, o); break;
      case 2: ring_direct<N, 2, MEAN>(x, d, lds, partial, o); break;
      default: ring_direct<N, 3, MEAN>(x, d, lds, partial, o); break;
    }
  }
}

// ---------------------------------------------------------------------------
// The guess: workgroup r makes Multi-Krum's selection on the kGuessRun
// coordinates from r * (d / kGuessRuns) on.
template <int N>
__global__ __launch_bounds__(kBlock) void k_guess(const float* __restrict__ x, int64_t d, int f,
                                                  int m, uint64_t* __restrict__ guess) {
  constexpr int P = N * (N - 1) / 2, W = kGuessRun / kBlock;
  static_assert(W == 4, "one 16-byte load per row and lane");
  __shared__ float part[kBlock / 64][P];
  __shared__ double esum[P];
  const int64_t c = static_cast<int64_t>(blockIdx.x) * (d / kGuessRuns) + threadIdx.x * W;
  float v[N][W], acc[P];
#pragma unroll
  for (int p = 0; p < P; ++p) acc[p] = 0.0f;
  direct_load<N, W>(MatrixRows{x, d}, c, d, v);
  direct_add<N, W>(v, acc);
  // the pairs' sums in fp32: a guess needs no more
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  using WS = WaveSums<64, float>;
#pragma unroll
  for (int base = 0; base < P; base += 64) {
    float t[64];
#pragma unroll
    for (int q = 0; q < 64; ++q) t[q] = base + q < P ? acc[base + q < P ? base + q : 0] : 0.0f;
    const float s = WS::run(t, lane);
    const int p = base + WS::index(lane);
    if (p < P) part[wave][p] = s;
  }
  __syncthreads();
  for (int p = threadIdx.x; p < P; p += kBlock)
    esum[p] = static_cast<double>((part[0][p] + part[1][p]) + (part[2][p] + part[3][p]));
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const uint64_t mask = krum_mask_wave<N>(esum, f, m);
  if (threadIdx.x == 0) guess[blockIdx.x] = mask;
}

// The mean after the selection (enqueue_mean_after). A workgroup covers
// kAfterChunks times 1,024 coordinates: with more of them a right guess, which
// leaves the workgroups nothing to do but read it, costs less (25.6 M
// coordinates: 19, 10 and 6 us with 1, 2 and 4), and a wrong one more (the
// mean of 7 rows: 132, 136 and 144 us).
constexpr int kAfterChunks = 2;

// SUMS: where no guess was agreed on, the column sums are there.
template <bool SUMS>
__global__ __launch_bounds__(kBlock) void k_mean_after(const float* __restrict__ x, int n,
                                                       int64_t d,
                                                       const int32_t* __restrict__ sel,
                                                       RingOut o) {
  uint64_t mask;
  const bool guessed = guess_agrees(o.guess, &mask);
  const uint64_t chosen = rows_mask(sel, o.m, n);
  if (guessed && chosen == mask) return;
  const MatrixRows src{x, d};
  int64_t c = (static_cast<int64_t>(blockIdx.x) * kAfterChunks * kBlock + threadIdx.x) * 4;
  for (int k = 0; k < kAfterChunks && c < d; ++k, c += 4 * kBlock) {
    if (SUMS && !guessed) complement_at<4>(src, n, d, sel, o.m, chosen, o.colsum, c, o.out);
    else mean_at<4>(src, d, ListedRows{sel, n}, o.m, c, o.out);
  }
}

template <int N>
hipError_t launch_ring(const float* x, const DistPlan& p, double* partial, const RingMean* mean,
                       hipStream_t s) {
  const RingOut o = mean ? RingOut{mean->guess, mean->colsum, mean->out, mean->m} : RingOut{};
  if constexpr (N >= kGuessMinN && N <= kGuessMaxN) {
    if (mean) {
      launch("dist_ring_mean", k_dist_ring<N, true>, dim3(static_cast<unsigned>(p.tiles)),
             dim3(kRingThreads), 0, s, x, p.d, partial, o);
      return hipGetLastError();
    }
  }
  if (mean) return hipErrorInvalidValue;
  launch("dist_ring", k_dist_ring<N, false>, dim3(static_cast<unsigned>(p.tiles)),
         dim3(kRingThreads), 0, s, x, p.d, partial, o);
  return hipGetLastError();
}

template <int N>
hipError_t ring_dispatch(const float* x, const DistPlan& p, double* partial, const RingMean* mean,
                         hipStream_t s) {
  if constexpr (N > kDirectMaxNLimit) {
    return hipErrorInvalidValue;
  } else {
    if (p.n == N) return launch_ring<N>(x, p, partial, mean, s);
    return ring_dispatch<N + 1>(x, p, partial, mean, s);
  }
}

template <int N>
hipError_t guess_dispatch(const float* x, int n, int64_t d, int f, int m, uint64_t* guess,
                          hipStream_t s) {
  if constexpr (N > kGuessMaxN) {
    return hipErrorInvalidValue;
  } else {
    if (n != N) return guess_dispatch<N + 1>(x, n, d, f, m, guess, s);
    launch("guess", k_guess<N>, dim3(kGuessRuns), dim3(kBlock), 0, s, x, d, f, m, guess);
    return hipGetLastError();
  }
}

template <int N>
constexpr int stage_of(int n) {
  if constexpr (N > kDirectMaxNLimit) return 0;
  else return n == N ? RingShape<N>::STAGE : stage_of<N + 1>(n);
}

}  // namespace

int ring_stage(int n) { return stage_of<2>(n); }

// The ring form has a longer start and end than the register form (one
// workgroup per CU: the first loads' latency, then one reduction over all
// pairs, with nothing beside them), and streams faster in between. Whole calls
// of garfield_pairwise_sqdist on N(0, 1) rows, ring against register form: n = 2
// 16.7 against 16.9 us at 8.4 M coordinates and 26.1 against 28.1 at 16.8 M;
// n = 5 32.5 against 33.0 and 57.5 against 60.7; n = 7 42.7 against 45.2 and
// 77.1 against 84.1; n = 12 67.4 against 77.6 and 128 against 150; n = 11's pass
// alone at 6 M 43.4 against 42.2. n = 16 31.2 against 32.8 us at 2.1 M and 89.5
// against 114 at 8.4 M; n = 20 38.8 against 41.9 and 124 against 143, its pass
// alone at 1.5 M 29.1 against 25.1.
bool ring_pays(int n, int64_t d) {
  if (n < 2 || n > kDirectMaxNLimit || d > int64_t{1} << 38) return false;
  return d >= int64_t{1} << (n >= 16 ? 21 : 23);
}

// A guess costs its launch and the look at it afterwards (4 to 10 us), and
// where the samples agree it saves a pass over m rows. Where they disagree
// nothing is saved, and the line is where the ring form's faster distance pass
// still makes up for it. Multi-Krum with m = n - f, whole calls in us in the
// register form without a guess, then in the ring form without one, with one
// the samples disagree on (N(0, 1) rows) and with a right one (f outliers):
//                          d = 8.4 M              d = 25.6 M
//   n =  5, f = 1    63.2  61.8  66.4  48.1    171  167  171  122
//   n =  7, f = 2    80.7  78.3  83.2  60.9    223  214  221  159
//   n =  8, f = 1    92.3  85.4  89.9  68.9    254  235  238  180
//   n = 11, f = 2     120   109   113  86.2    331  311  313  242
//   n = 14, f = 2     172   157   169   122    504  452  467  327
//   n = 17, f = 3     213   189   199   153    616  535  550  415
//   n = 20, f = 4     251   220   234   194    735  645  667  539
// Up to 10 rows the ring form gains too little below 2^24, except on calls with
// column sums (2m > n + 4) and on those that keep every row, whose guess is
// never wrong. (In a burst of 21 calls, under the clock's dip at its start, 15 to
// 19 rows of 10 M coordinates take 3 % longer with a wrong guess than in the
// register form, 7 rows 2 % longer, 11 rows 4 % less.) A selection of fewer than
// n - f rows among rows alike is never guessed right: n = 17, m = 8 157 us with a
// guess and 151 without, 176 in the register form.
bool guess_pays(int n, int64_t d, int f, int m, const float* out) {
  if (n < kGuessMinN || n > kGuessMaxN || n < 2 * f + 3 || m < 2 || !out || load_width(out) != 4)
    return false;
  const bool sure = n >= 11 || m == n || 2 * m > n + 4;
  return d >= int64_t{1} << (sure ? 23 : 24) && d <= int64_t{1} << 38;
}

hipError_t enqueue_distances_ring(const float* x, const DistPlan& p, double* partial,
                                  const RingMean* mean, hipStream_t s) {
  return ring_dispatch<2>(x, p, partial, mean, s);
}

hipError_t enqueue_guess(const float* x, int n, int64_t d, int f, int m, uint64_t* guess,
                         hipStream_t s) {
  return guess_dispatch<kGuessMinN>(x, n, d, f, m, guess, s);
}

hipError_t enqueue_mean_after(const float* x, int n, int64_t d, const int32_t* sel,
                              const RingMean& mean, hipStream_t s) {
  const int64_t per = int64_t{4} * kBlock * kAfterChunks;
  const int64_t groups = (d + per - 1) / per;
  if (groups > 0x7fffffff) return hipErrorInvalidValue;
  launch("mean_after", mean.colsum ? k_mean_after<true> : k_mean_after<false>,
         dim3(static_cast<unsigned>(groups)), dim3(kBlock), 0, s, x, n, d, sel,
         RingOut{mean.guess, mean.colsum, mean.out, mean.m});
  return hipGetLastError();
}

}  // namespace garfield

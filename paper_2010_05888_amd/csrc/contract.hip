// Contraction steps (decentralized learning, Section 5: each node repeatedly
// aggregates the vectors it receives from its peers). All N nodes' vectors are
// the rows of one N x d matrix x; node v's peers are peers[v*q .. v*q+q-1].
// One step writes every node's aggregate of its peers to row v of y. The
// selection kernel (k_peer_select) runs one workgroup per node on the
// distances of all N rows; the kernels below then aggregate every node in one
// launch. Mean and Median stage a tile of all N rows in LDS (each input value
// read from HBM once, in runs of 1 KB or more) and compute every node's output
// for that tile from it, with what the nodes share done once for up to 32 of
// them (k_mean_shared, k_median_shared); Bulyan, bound by its per-node
// arithmetic rather than its loads, takes one workgroup per (tile, node), see
// node_grid. The results are the single-rule kernels' own, bit for bit.

#include "aggregate_body.h"
#include "internal.h"
#include "timing.h"

namespace garfield {

namespace {

// Workgroups of a step: every (tile, node) pair, mapped so that the nodes of one
// tile run back to back on one XCD. Workgroups are dispatched round-robin over
// the 8 XCDs; XCD x takes tiles x, x + 8, ..., and for each of them all nodes
// in turn, with ordinary (L2-allocating) loads, so the rows the nodes share
// come from that XCD's L2 after the first node read them. (Staging a tile of
// all rows in LDS and looping over the nodes in one workgroup was slower: the
// stage leaves one or two workgroups per CU.)
constexpr int kXcds = 8;

int64_t tiles_for(int64_t d, int w) {
  return (d + static_cast<int64_t>(kBlock) * w - 1) / (static_cast<int64_t>(kBlock) * w);
}

dim3 node_grid(int64_t tiles, int nodes) {
  const int64_t padded = (tiles + kXcds - 1) / kXcds * kXcds;
  return dim3(static_cast<unsigned>(padded * nodes));
}

// (tile, node) of this workgroup; tile may be past the last one (padding).
__device__ __forceinline__ void node_tile(int nodes, int64_t* tile, int* v) {
  const int64_t b = blockIdx.x;
  const int64_t j = b / kXcds;
  *tile = (j / nodes) * kXcds + b % kXcds;
  *v = static_cast<int>(j % nodes);
}

// LDS tile: coordinates c0 .. c0+255 of all n rows, row r at tile[r * 256].
// Wave w loads rows w, w + 4, ... with one 16-byte nontemporal load per lane
// (1 KB of a row per instruction), all of its rows before any store to LDS.
constexpr int kTileCoords = kBlock;
constexpr int kTileRowsPerWave = kNmax / 4;

__device__ __forceinline__ void stage_tile(const float* __restrict__ x, int n, int64_t d,
                                           int64_t c0, float* __restrict__ tile) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c = c0 + 4 * lane;
  float v[kTileRowsPerWave][4];
#pragma unroll
  for (int u = 0; u < kTileRowsPerWave; ++u) {
    const int r = wave + 4 * u;  // wave-uniform
    if (r < n) {
      const float* p = x + static_cast<int64_t>(r) * d + c;
      if (c + 4 <= d) load_w<4>(p, v[u]); else load_w_tail<4>(p, d - c, v[u]);
    }
  }
#pragma unroll
  for (int u = 0; u < kTileRowsPerWave; ++u) {
    const int r = wave + 4 * u;
    if (r < n) {
      float* q = tile + r * kTileCoords + 4 * lane;
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] = v[u][e];
    }
  }
  __syncthreads();
}

// The nodes' row lists, as LDS offsets into the tile (row * 256), after the
// tile in dynamic LDS.
__device__ __forceinline__ int32_t* stage_offsets(const int32_t* __restrict__ rows, int count,
                                                  int n, float* tile) {
  int32_t* off = reinterpret_cast<int32_t*>(tile + n * kTileCoords);
  for (int i = threadIdx.x; i < count; i += kBlock)
    off[i] = static_cast<int32_t>(row_of(rows, i, n)) * kTileCoords;
  return off;
}

// Node v's output at coordinate c0 + t: the mean of its k rows (rows[v*k ..],
// fp64 sum in the order listed, one rounding), for every node; two nodes'
// sums at a time, so that two chains of additions are in flight.
__global__ __launch_bounds__(kBlock) void k_mean_nodes(const float* __restrict__ x, int n,
                                                       int64_t d, int nodes,
                                                       const int32_t* __restrict__ rows, int k,
                                                       float* __restrict__ y) {
  extern __shared__ float tile[];
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kTileCoords;
  const int32_t* off = stage_offsets(rows, nodes * k, n, tile);
  stage_tile(x, n, d, c0, tile);  // ends with a barrier
  const int t = threadIdx.x;
  const int64_t c = c0 + t;
  if (c >= d) return;
  const double count = static_cast<double>(k);
  int v = 0;
  for (; v + 2 <= nodes; v += 2) {
    const int32_t* o0 = off + v * k;
    const int32_t* o1 = o0 + k;
    double a0 = 0.0, a1 = 0.0;
#pragma unroll 4
    for (int i = 0; i < k; ++i) {
      a0 += static_cast<double>(tile[o0[i] + t]);
      a1 += static_cast<double>(tile[o1[i] + t]);
    }
    __builtin_nontemporal_store(static_cast<float>(a0 / count), y + static_cast<int64_t>(v) * d + c);
    __builtin_nontemporal_store(static_cast<float>(a1 / count),
                                y + static_cast<int64_t>(v + 1) * d + c);
  }
  if (v < nodes) {
    const int32_t* o0 = off + v * k;
    double a0 = 0.0;
#pragma unroll 4
    for (int i = 0; i < k; ++i) a0 += static_cast<double>(tile[o0[i] + t]);
    __builtin_nontemporal_store(static_cast<float>(a0 / count), y + static_cast<int64_t>(v) * d + c);
  }
}

// Node v's output: the median of its K rows (the selection network of the
// single-rule median), for every node.
template <int K>
__global__ __launch_bounds__(kBlock) void k_median_nodes(const float* __restrict__ x, int n,
                                                         int64_t d, int nodes,
                                                         const int32_t* __restrict__ rows,
                                                         float* __restrict__ y) {
  using Net = MedianNet<K>;
  extern __shared__ float tile[];
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kTileCoords;
  const int32_t* off = stage_offsets(rows, nodes * K, n, tile);
  stage_tile(x, n, d, c0, tile);  // ends with a barrier
  const int t = threadIdx.x;
  const int64_t c = c0 + t;
  if (c >= d) return;
  for (int v = 0; v < nodes; ++v) {
    const int32_t* ov = off + v * K;
    float a[K];
#pragma unroll
    for (int i = 0; i < K; ++i) a[i] = tile[ov[i] + t];
    Net::run(a);
    float o;
    if constexpr (K % 2 == 1) {
      o = a[Net::LO];
    } else {  // mean of the two middle values, exact in fp64, rounded once
      o = static_cast<float>((static_cast<double>(a[Net::LO]) + static_cast<double>(a[Net::HI])) *
                             0.5);
    }
    __builtin_nontemporal_store(o, y + static_cast<int64_t>(v) * d + c);
  }
}

// ---------------------------------------------------------------------------
// Few rows (n <= kSharedMaxRows): what the nodes share is done once per
// coordinate, from registers. A workgroup stages kSharedCoords coordinates of
// all N rows in LDS and every lane takes two of them, so each output row is
// written in 512-byte runs per wave.
//
// Mean: the lane converts its N values to fp64 once and, for every node, adds
// the rows in ascending order, each times 1 or 0 as the node's mask says (an
// exact product; the weights are scalars formed beside the vector work). The
// form above reads every listed value from LDS again, with its offset, and
// converts it: 28 LDS reads and 42 vector instructions per node of 14 rows,
// against 20 multiply-adds here at N = 20. (A uniform branch per row in place
// of the weight took 711 us where this takes 420 and the form above 548: n = 20
// nodes of 11.2 M coordinates, 14 rows each.)
//
// Median: the lane sorts its N values once, and a node that hears all but X of
// them takes the middle of what is left when its X absent values are removed
// from the sorted row: with those in ascending order e[1..X], the rank-t value
// of the rest is s[t] if e[1] > s[t], else s[t + 1] if e[2] > s[t + 1], and so
// on. X LDS reads, a sort of X values and 2 X selects per node and rank, where
// the network over q values took q reads and about 6 q instructions: 827 -> 410
// us for n = 20 nodes of 11.2 M coordinates and 17 peers.
//
// Both then run at 4.3 TB/s of rows read and rows written, the rate of a copy
// on this chip (4.6); at 32 nodes the vector work per node bounds them again.
//
// A node whose list repeats a row (its mask has fewer rows) takes its listed
// rows in order, and so do all nodes of a wave that holds what the shared work
// would carry over from rows a node does not hear: for the mean an infinity or
// NaN (a weight of 0 would not leave those out), for the median a NaN (the
// networks' minima and maxima drop it, and another value stands there twice).
constexpr int kSharedMaxRows = 32;
constexpr int kSharedCoords = 2 * kBlock;
constexpr int kSharedMaxAbsent = 6;
constexpr int64_t kSharedMinCoords = int64_t{1} << 18;  // two workgroups per CU

// Coordinates c0 .. c0 + kSharedCoords - 1 of all N rows into LDS, row r at
// tile[r * kSharedCoords]; those at or beyond d read as 0. Wave w loads 1 KB
// pieces w, w + 4, ..., all of them before any store to LDS. No barrier.
template <int N>
__device__ __forceinline__ void stage_rows(const float* __restrict__ x, int64_t d, int64_t c0,
                                           float* __restrict__ tile) {
  constexpr int PARTS = kSharedCoords / 256, TOTAL = N * PARTS, PER = (TOTAL + 3) / 4;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (c0 + kSharedCoords <= d) {  // uniform: a whole tile
    f4 v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int j = wave + 4 * u;  // wave-uniform
      if (u < TOTAL / 4 || j < TOTAL)
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(
            x + static_cast<int64_t>(j / PARTS) * d + c0 + (j % PARTS) * 256 + 4 * lane));
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int j = wave + 4 * u;
      if (u < TOTAL / 4 || j < TOTAL) *reinterpret_cast<f4*>(tile + j * 256 + 4 * lane) = v[u];
    }
  } else {
    for (int i = threadIdx.x; i < N * kSharedCoords; i += kBlock) {
      const int64_t c = c0 + i % kSharedCoords;
      tile[i] = c < d ? x[static_cast<int64_t>(i / kSharedCoords) * d + c] : 0.0f;
    }
  }
}

__device__ __forceinline__ void store_pair(float* __restrict__ row, int64_t c, int64_t d, float a,
                                           float b) {
  const float o[2] = {a, b};
  if (c + 2 <= d) store_w<2>(row + c, o);
  else if (c < d) row[c] = a;
}

template <int N>
__global__ __launch_bounds__(kBlock) void k_mean_shared(const float* __restrict__ x, int64_t d,
                                                        int nodes,
                                                        const int32_t* __restrict__ rows, int k,
                                                        float* __restrict__ y) {
  __shared__ __attribute__((aligned(16))) float tile[N * kSharedCoords];
  __shared__ uint32_t masks[kNmax];  // 0: the node's list repeats a row
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kSharedCoords;
  if (static_cast<int>(threadIdx.x) < nodes) {
    uint32_t m = 0;
    for (int i = 0; i < k; ++i) m |= 1u << row_of(rows + threadIdx.x * k, i, N);
    masks[threadIdx.x] = __builtin_popcount(m) == k ? m : 0;
  }
  stage_rows<N>(x, d, c0, tile);
  __syncthreads();
  const int64_t c = c0 + 2 * threadIdx.x;
  double a[N], b[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const f2 t = *reinterpret_cast<const f2*>(tile + i * kSharedCoords + 2 * threadIdx.x);
    a[i] = static_cast<double>(t.x);
    b[i] = static_cast<double>(t.y);
  }
  double z = 0.0;  // NaN if any value is not finite
#pragma unroll
  for (int i = 0; i < N; ++i) z = __builtin_fma(a[i], 0.0, __builtin_fma(b[i], 0.0, z));
  const bool finite = __ballot(__builtin_isnan(z)) == 0;
  const double count = static_cast<double>(k), inv = 1.0 / count;
  for (int v = 0; v < nodes; ++v) {
    const uint32_t m = __builtin_amdgcn_readfirstlane(masks[v]);
    double s0 = 0.0, s1 = 0.0;
    if (m && finite) {  // uniform
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const double w = (m >> i) & 1 ? 1.0 : 0.0;
        s0 = __builtin_fma(a[i], w, s0);
        s1 = __builtin_fma(b[i], w, s1);
      }
    } else {
      for (int i = 0; i < k; ++i) {
        const float* p = tile + row_of(rows + v * k, i, N) * kSharedCoords + 2 * threadIdx.x;
        s0 += static_cast<double>(p[0]);
        s1 += static_cast<double>(p[1]);
      }
    }
    store_pair(y + static_cast<int64_t>(v) * d, c, d, static_cast<float>(mean_of(s0, count, inv)),
               static_cast<float>(mean_of(s1, count, inv)));
  }
}

// e <= at in the order the networks sort by (their minimum takes -0 before +0,
// where a comparison of floats calls the two equal): the order of the bits, whose
// magnitudes count downwards where at is negative.
__device__ __forceinline__ bool sorts_to(float e, float at) {
  const int32_t b = __float_as_int(at), flip = (b >> 31) & 0x7fffffff;
  return (__float_as_int(e) ^ flip) <= (b ^ flip);
}

// The rank-T value of the N sorted values s (rank r at s[Net::reg(r)]) without
// the X values e (ascending).
template <int N, int X, int T>
__device__ __forceinline__ float rank_without(const float* s, const float* e) {
  using Net = SortNet<N>;
  float r = s[Net::reg(T + X)];
#pragma unroll
  for (int k = X - 1; k >= 0; --k) {
    const float at = s[Net::reg(T + k)];
    r = sorts_to(e[k], at) ? r : at;
  }
  return r;
}

// The median of the N - X values left of s (as above).
template <int N, int X>
__device__ __forceinline__ float median_without(const float* s, float* e) {
  constexpr int Q = N - X;
  if constexpr (X >= 2) {
    float t[X];
#pragma unroll
    for (int k = 0; k < X; ++k) t[k] = e[k];
    SortNet<X>::run(t);
#pragma unroll
    for (int k = 0; k < X; ++k) e[k] = t[SortNet<X>::reg(k)];
  }
  const float lo = rank_without<N, X, (Q - 1) / 2>(s, e);
  if constexpr (Q % 2 == 1) {
    return lo;
  } else {  // mean of the two middle values, exact in fp64, rounded once
    const float hi = rank_without<N, X, Q / 2>(s, e);
    return static_cast<float>((static_cast<double>(lo) + static_cast<double>(hi)) * 0.5);
  }
}

template <int N, int X>
__global__ __launch_bounds__(kBlock) void k_median_shared(const float* __restrict__ x, int64_t d,
                                                          int nodes,
                                                          const int32_t* __restrict__ rows,
                                                          float* __restrict__ y) {
  constexpr int Q = N - X;
  constexpr int XP = X <= 4 ? 4 : 8;  // offsets per node, read 16 bytes at a time
  __shared__ __attribute__((aligned(16))) float tile[N * kSharedCoords];
  __shared__ __attribute__((aligned(16))) int32_t absent[kNmax * XP];  // offsets into tile
  __shared__ int whole[kNmax];  // the node's list holds Q rows
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kSharedCoords;
  if (static_cast<int>(threadIdx.x) < nodes) {
    uint32_t m = 0;
    for (int i = 0; i < Q; ++i) m |= 1u << row_of(rows + threadIdx.x * Q, i, N);
    const bool ok = __builtin_popcount(m) == Q;
    whole[threadIdx.x] = ok;
    uint32_t rest = ok ? ~m & (N == 32 ? ~0u : (1u << N) - 1) : 0;
    for (int k = 0; k < XP; ++k, rest &= rest - 1)
      absent[threadIdx.x * XP + k] = rest ? __builtin_ctz(rest) * kSharedCoords : 0;
  }
  stage_rows<N>(x, d, c0, tile);
  __syncthreads();
  const int64_t c = c0 + 2 * threadIdx.x;
  const float* mine = tile + 2 * threadIdx.x;
  float s0[N], s1[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const f2 t = *reinterpret_cast<const f2*>(mine + i * kSharedCoords);
    s0[i] = t.x;
    s1[i] = t.y;
  }
  bool nan = false;
#pragma unroll
  for (int i = 0; i < N; ++i) nan |= __builtin_isunordered(s0[i], s1[i]);
  const bool ordered = __ballot(nan) == 0;
  SortNet<N>::run(s0);
  SortNet<N>::run(s1);
  for (int v = 0; v < nodes; ++v) {
    float o0, o1;
    if (ordered && __builtin_amdgcn_readfirstlane(whole[v])) {  // uniform
      float e0[X > 0 ? X : 1], e1[X > 0 ? X : 1];
#pragma unroll
      for (int k = 0; k < X; ++k) {
        const f2 t = *reinterpret_cast<const f2*>(mine + absent[v * XP + k]);
        e0[k] = t.x;
        e1[k] = t.y;
      }
      o0 = median_without<N, X>(s0, e0);
      o1 = median_without<N, X>(s1, e1);
    } else {
      using Net = MedianNet<Q>;
      float a[Q], b[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const float* p = mine + row_of(rows + v * Q, i, N) * kSharedCoords;
        a[i] = p[0];
        b[i] = p[1];
      }
      Net::run(a);
      Net::run(b);
      if constexpr (Q % 2 == 1) {
        o0 = a[Net::LO];
        o1 = b[Net::LO];
      } else {
        o0 = static_cast<float>((static_cast<double>(a[Net::LO]) + static_cast<double>(a[Net::HI])) * 0.5);
        o1 = static_cast<float>((static_cast<double>(b[Net::LO]) + static_cast<double>(b[Net::HI])) * 0.5);
      }
    }
    store_pair(y + static_cast<int64_t>(v) * d, c, d, o0, o1);
  }
}

unsigned shared_grid(int64_t d) {
  return static_cast<unsigned>((d + kSharedCoords - 1) / kSharedCoords);
}

template <int N>
hipError_t mean_shared_dispatch(const float* x, int n, int64_t d, int nodes, const int32_t* rows,
                                int k, float* y, hipStream_t s) {
  if constexpr (N > kSharedMaxRows) {
    return hipErrorInvalidValue;
  } else {
    if (n != N) return mean_shared_dispatch<N + 1>(x, n, d, nodes, rows, k, y, s);
    launch("mean_nodes", k_mean_shared<N>, dim3(shared_grid(d)), dim3(kBlock), 0, s, x, d, nodes,
           rows, k, y);
    return hipGetLastError();
  }
}

template <int N, int X>
hipError_t median_shared_absent(const float* x, int64_t d, int nodes, const int32_t* rows, int q,
                                float* y, hipStream_t s) {
  if constexpr (X > kSharedMaxAbsent || 3 * X >= N) {
    return hipErrorInvalidValue;
  } else {
    if (q != N - X) return median_shared_absent<N, X + 1>(x, d, nodes, rows, q, y, s);
    launch("median_nodes", k_median_shared<N, X>, dim3(shared_grid(d)), dim3(kBlock), 0, s, x, d,
           nodes, rows, y);
    return hipGetLastError();
  }
}

template <int N>
hipError_t median_shared_dispatch(const float* x, int n, int64_t d, int nodes,
                                  const int32_t* rows, int q, float* y, hipStream_t s) {
  if constexpr (N > kSharedMaxRows) {
    return hipErrorInvalidValue;
  } else {
    if (n != N) return median_shared_dispatch<N + 1>(x, n, d, nodes, rows, q, y, s);
    return median_shared_absent<N, 0>(x, d, nodes, rows, q, y, s);
  }
}

unsigned tile_grid(int64_t d) {
  return static_cast<unsigned>((d + kTileCoords - 1) / kTileCoords);
}
// The tile and the nodes' row offsets (count entries).
size_t tile_bytes(int n, int count) {
  return static_cast<size_t>(n) * kTileCoords * sizeof(float) + count * sizeof(int32_t);
}

template <int T, int W>
__global__ __launch_bounds__(kBlock) void k_bulyan_nodes(const float* __restrict__ x, int n,
                                                         int64_t d, int nodes,
                                                         const int32_t* __restrict__ sel,
                                                         int beta, float* __restrict__ y) {
  __shared__ float sorted[T * kBlock];
  int64_t tile;
  int v;
  node_tile(nodes, &tile, &v);
  const int64_t c = (tile * kBlock + threadIdx.x) * W;
  if (c < d)
    bulyan_at<T, W, false>(MatrixRows{x, d}, d, ListedRows{sel + static_cast<int64_t>(v) * T, n},
                           beta, c, sorted + threadIdx.x, y + static_cast<int64_t>(v) * d);
}

// Bulyan's width as the single-rule kernel chooses it for float-aligned rows
// (the entry point requires those): the T x W values of a lane must fit the
// registers of two waves per SIMD.
template <int K>
hipError_t median_nodes_dispatch(int k, const float* x, int n, int64_t d, int nodes,
                                 const int32_t* rows, float* y, hipStream_t s) {
  if constexpr (K > kNmax) {
    return hipErrorInvalidValue;
  } else {
    if (k != K) return median_nodes_dispatch<K + 1>(k, x, n, d, nodes, rows, y, s);
    launch("median_nodes", k_median_nodes<K>, dim3(tile_grid(d)), dim3(kBlock),
           static_cast<uint32_t>(tile_bytes(n, nodes * K)), s, x, n, d, nodes, rows, y);
    return hipGetLastError();
  }
}

template <int T>
hipError_t bulyan_nodes_dispatch(int theta, int beta, const float* x, int n, int64_t d,
                                 int nodes, const int32_t* sel, float* y, hipStream_t s) {
  if constexpr (T > kNmax) {
    return hipErrorInvalidValue;
  } else {
    if (theta != T)
      return bulyan_nodes_dispatch<T + 1>(theta, beta, x, n, d, nodes, sel, y, s);
    constexpr int W = T <= 24 ? 4 : (T <= 48 ? 2 : 1);
    launch("bulyan_nodes", k_bulyan_nodes<T, W>, node_grid(tiles_for(d, W), nodes), dim3(kBlock),
           0, s, x, n, d, nodes, sel, beta, y);
    return hipGetLastError();
  }
}

}  // namespace

namespace {

// Where the shared mean is the faster form. Its work per node grows with n, the
// other's with k, so it takes most of the rows to be chosen; and it holds two
// workgroups per CU from n = 20 on, in step with each other, so that short
// inputs end in a round that leaves the chip half idle. How many times as fast
// as the other form it is (the kernels alone, every node of n hearing all):
//                 d = 330 K   400 K   700 K   1.5 M   2.5 M    4 M   11.2 M
//   n =  9, k = 4    0.98     1.07    1.12    1.10    1.05    1.10    1.06
//   n = 12, k = 6    1.07     1.03    1.22    1.09    1.00    1.12    1.07
//   n = 16, k = 8    0.98     0.92    0.86    0.83    1.03    1.08    1.10
//           k = 11   1.12     1.07    1.03    0.98    1.23    1.28    1.28
//           k = 14   1.18     1.13    1.08    1.05    1.33    1.41    1.41
//   n = 20, k = 10   0.71     0.77    0.86    0.80    0.98    1.06    1.11
//           k = 13   0.77     0.81    0.90    0.87    1.07    1.19    1.22
//           k = 17   0.85     0.91    1.04    1.01    1.22    1.35    1.42
//   n = 28, k = 14   0.68     0.74    0.78    0.76    0.82    0.89    0.97
//           k = 19   0.80     0.89    0.93    0.92    0.99    1.08    1.19
//           k = 24   0.86     0.95    1.01    1.03    1.11    1.21    1.33
//   n = 32, k = 8    0.50     0.56    0.58    0.57    0.58    0.64    0.76
bool mean_shared_pays(int n, int k, int64_t d) {
  if (n > kSharedMaxRows || d < kSharedMinCoords) return false;
  if (d < int64_t{1} << 19) return n <= 18 && 6 * k >= 5 * n;
  if (n <= 9) return true;
  if (n <= 12) return 2 * k >= n;
  if (d < int64_t{1} << 21) return 6 * k >= 5 * n;
  if (d < int64_t{1} << 23) return 3 * k >= 2 * n;
  return 2 * k > n;
}

}  // namespace

hipError_t enqueue_mean_nodes(const float* x, int n, int64_t d, int nodes, const int32_t* rows,
                              int k, bool ascending, float* y, hipStream_t s) {
  if (d == 0 || nodes == 0) return hipSuccess;
  if (ascending && mean_shared_pays(n, k, d))
    return mean_shared_dispatch<1>(x, n, d, nodes, rows, k, y, s);
  launch("mean_nodes", k_mean_nodes, dim3(tile_grid(d)), dim3(kBlock),
         static_cast<uint32_t>(tile_bytes(n, nodes * k)), s, x, n, d, nodes, rows, k, y);
  return hipGetLastError();
}

namespace {

// Where the shared median is the faster form. It gains with every row a node
// hears and loses with every one it does not, and its workgroups of 512
// coordinates are too few for short inputs of few rows. How many times as fast
// as the network over each node's values it is (the kernels alone):
//                    d = 262 K   330 K   450 K   800 K   1.2 M   2.1 M   4 M   11.2 M
//   n =  7, 1 absent    0.90     0.89    1.02    1.21    1.08    1.15   1.17    1.11
//   n = 10, 3 absent    0.81     0.95    0.90    1.00    0.98    0.92   1.03    1.03
//   n = 11, 3 absent    0.89     0.96    0.97    0.87    0.94    0.93   1.07    1.14
//   n = 13, 4 absent    1.02     0.95    0.96    0.94    0.93    0.95   1.10    1.12
//   n = 17, 4 absent    1.24     1.17    1.18    1.31    1.30    1.33   1.60    1.64
//   n = 17, 5 absent    0.92     0.89    0.86    0.95    0.98    1.06   1.13    1.18
//   n = 20, 6 absent    1.02     0.99    0.92    1.02    1.02    1.12   1.16    1.21
//   n = 22, 6 absent    1.14     1.09    1.02    1.15    1.19    1.28   1.31    1.36
bool median_shared_pays(int n, int k, int64_t d) {
  const int absent = n - k;
  if (n > kSharedMaxRows || absent > kSharedMaxAbsent || 3 * absent >= n) return false;
  if (11 * absent >= 3 * n && n < 21) return d >= int64_t{1} << (n < 16 ? 22 : 21);
  return d >= (n < 14 ? 3 * kSharedMinCoords / 2 : kSharedMinCoords);
}

}  // namespace

hipError_t enqueue_median_nodes(const float* x, int n, int64_t d, int nodes, const int32_t* rows,
                                int k, float* y, hipStream_t s) {
  if (d == 0 || nodes == 0) return hipSuccess;
  if (median_shared_pays(n, k, d))
    return median_shared_dispatch<1>(x, n, d, nodes, rows, k, y, s);
  return median_nodes_dispatch<1>(k, x, n, d, nodes, rows, y, s);
}

hipError_t enqueue_bulyan_nodes(const float* x, int n, int64_t d, int nodes, int q, int f,
                                const int32_t* sel, float* y, hipStream_t s) {
  if (d == 0 || nodes == 0) return hipSuccess;
  const int theta = q - 2 * f;
  return bulyan_nodes_dispatch<1>(theta, theta - 2 * f, x, n, d, nodes, sel, y, s);
}

}  // namespace garfield

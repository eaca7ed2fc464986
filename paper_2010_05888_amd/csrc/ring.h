// Rows streamed through an LDS ring. A workgroup of eight waves walks stages
// of STAGE consecutive coordinates of N rows; the rows of a stage go from HBM
// straight into a slot of the ring (global_load_lds, 16 bytes a lane, 1 KB of
// one row per instruction), so the loads in flight take no registers and do
// not depend on how many waves the registers allow: one workgroup per CU keeps
// 80 to 120 KB in flight whatever its accumulators need. Rows start at any
// float (the instruction takes dword-aligned addresses), and in LDS every row
// of a slot is 16-byte aligned.
#pragma once

#include "device_common.h"
#include "internal.h"
#include "rows.h"

namespace garfield {

constexpr int kRingWaves = 8;
constexpr int kRingThreads = kRingWaves * 64;
constexpr int kLdsPerCu = 160 * 1024;

// LDS-only barrier: waits for this wave's LDS operations, then for every
// wave, and leaves vector-memory loads in flight (a __syncthreads() would also
// wait for those).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt unconstrained
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Wait until at most VM of this wave's vector-memory operations are in flight.
template <int VM>
__device__ __forceinline__ void wait_vm() {
  static_assert(VM >= 0 && VM < 64, "vmcnt has six bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (VM & 15) | ((VM >> 4) << 14));
  asm volatile("" ::: "memory");
}

// 16 bytes per lane from g (each lane its own address) to l + 16 * lane (l the
// same in every lane, 16-byte aligned).
__device__ __forceinline__ void load_to_lds(const float* g, float* l) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)g,
      (__attribute__((address_space(3))) void*)l, 16, 0, 2);  // nontemporal
}

// The stages of a launch over one row-major n x d matrix: entry i of this
// workgroup is stage slot + i * G. Workgroups are dealt to the 8 XCDs
// round-robin (block b to XCD b % 8), so slot (b % 8) * (G / 8) + b / 8 gives
// each XCD a contiguous run of stages, and neighbouring stages, which share
// the cache lines at the ends of their row runs, meet in one XCD's L2. (A
// bijection on [0, G) when 8 divides G; other grids keep b.)
__device__ __forceinline__ int64_t xcd_slot() {
  const int64_t b = blockIdx.x, G = gridDim.x;
  if (G % 8 != 0) return b;
  return (b % 8) * (G / 8) + b / 8;
}

// Ring of N rows: STAGE coordinates per stage, and as many slots as hold about
// 96 KB in flight beside the stage being read and the next one.
template <int N>
struct RingShape {
  static constexpr int STAGE = N <= 10 ? 1024 : 512;
  static constexpr int SLOT = N * STAGE;  // floats per slot
  static constexpr int FIT = kLdsPerCu / (SLOT * 4);
  static constexpr int WANT = 3 + 96 * 1024 / (SLOT * 4);
  static constexpr int SLOTS = WANT < FIT ? WANT : FIT;
  static constexpr int AHEAD = SLOTS - 1;        // stages issued ahead of the one being read
  static constexpr int LOADS = SLOT / 256;       // 1 KB loads per stage
  static constexpr int PER = LOADS / kRingWaves; // of one wave, and one more
  static constexpr int MORE = LOADS % kRingWaves;  // in this many waves
  static constexpr int MAXPER = PER + (MORE != 0);
  static_assert(SLOTS >= 4, "a stage read, the next one landed, and two filling");
  static_assert((AHEAD - 1) * MAXPER < 64, "vmcnt has six bits");
};

// This lane's number, formed anew where it is used.
__device__ __forceinline__ uint32_t fresh_lane() {
  uint32_t lane;
  asm volatile(
      "v_mbcnt_lo_u32_b32 %0, -1, 0\n\t"
      "v_mbcnt_hi_u32_b32 %0, -1, %0"
      : "=v"(lane));
  return lane;
}

// A wave's share of a stage's loads: one pointer per load (wave-uniform; the
// lanes add 16 bytes each), all of which advance by the same `step` floats
// from one stage of the workgroup to its next.
template <int N>
struct RingLoads {
  using R = RingShape<N>;
  const float* p[R::MAXPER];

  template <class Src>
  __device__ __forceinline__ void start(const Src& src, int64_t c0, int wave) {
    constexpr int PARTS = R::STAGE / 256;
#pragma unroll
    for (int u = 0; u < R::MAXPER; ++u) {
      const int j = wave + u * kRingWaves;  // wave-uniform
      const int k = j < R::LOADS ? j : 0;
      p[u] = src.row(k / PARTS) + c0 + (k % PARTS) * 256;
    }
  }
  // Issue the next stage's loads into `slot`. No memory access written after
  // them is moved ahead of them: ring_wait counts the stores that follow a
  // stage's loads, and one that went first would leave it a store short, so that
  // a stage could be read before it has landed. (Nothing else keeps the order: the
  // rows are const and restrict, and the stores go elsewhere.)
  __device__ __forceinline__ void issue(float* slot, int64_t step, int wave, uint32_t lane) {
#pragma unroll
    for (int u = 0; u < R::MAXPER; ++u) {
      if (u < R::PER || wave < R::MORE)
        load_to_lds(p[u] + 4 * lane, slot + (wave + u * kRingWaves) * 256);
      p[u] += step;
    }
    asm volatile("" ::: "memory");
  }
};

// Wait for this wave's loads of all but the last LEFT stages issued (`steady`),
// else for all of them. STORES: vector stores this wave has issued, without
// exception, since the loads waited for (stores and loads leave the count in the
// order they were issued in, which is that of the source, see issue).
template <int N, int LEFT, int STORES = 0>
__device__ __forceinline__ void ring_wait(bool steady, int wave) {
  using R = RingShape<N>;
  constexpr int HI = LEFT * (R::PER + 1) + STORES, LO = LEFT * R::PER + STORES;
  if (!steady) wait_vm<0>();
  else if (R::MORE != 0 && wave < R::MORE) wait_vm<(HI < 63 ? HI : 63)>();
  else wait_vm<(LO < 63 ? LO : 63)>();
}

// v of the lane that the DPP control CTRL names, for this lane.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_word(uint32_t v) {
  return static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ float dpp_lane(float v) {
  return __uint_as_float(dpp_word<CTRL>(__float_as_uint(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_lane(double v) {
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
  const uint64_t lo = dpp_word<CTRL>(static_cast<uint32_t>(b));
  const uint64_t hi = dpp_word<CTRL>(static_cast<uint32_t>(b >> 32));
  return __longlong_as_double(static_cast<int64_t>((hi << 32) | lo));
}

// Sums over the 64 lanes of M (at most 64) values per lane, by a butterfly
// that halves the values kept at every step: lane l's result is the sum of
// value index(l). Lanes l and l ^ 15, then l ^ 7, l ^ 3 and l ^ 1 (mirrors and
// quad permutes, in the vector unit), then the rows of 16 exchange halves: at
// each step the two lanes hold the same values' partial sums and bit b of l
// (b = 3, 2, 1, 0, then 4, 5) says which half stays. The lanes meet in the
// same pairs whatever the value, so every value is summed by the same tree.
template <int M, class T>
struct WaveSums {
  static constexpr int LOG =
      M <= 1 ? 0 : (M <= 2 ? 1 : (M <= 4 ? 2 : (M <= 8 ? 3 : (M <= 16 ? 4 : (M <= 32 ? 5 : 6)))));
  static constexpr int P = 1 << LOG;
  static_assert(M <= 64, "at most a value per lane");
  static __host__ __device__ constexpr int bit(int step) { return step < 4 ? 3 - step : step; }

  template <int S>
  static __device__ __forceinline__ T across(T v) {
    if constexpr (S == 0) return dpp_lane<0x140>(v);       // row_mirror: l ^ 15
    else if constexpr (S == 1) return dpp_lane<0x141>(v);  // row_half_mirror: l ^ 7
    else if constexpr (S == 2) return dpp_lane<0x1B>(v);   // quad_perm [3, 2, 1, 0]: l ^ 3
    else if constexpr (S == 3) return dpp_lane<0xB1>(v);   // quad_perm [1, 0, 3, 2]: l ^ 1
    else return __shfl_xor(v, 1 << S, 64);                 // l ^ 16, l ^ 32
  }
  // its sizes compile-time, so that every value stays in a register
  template <int S>
  static __device__ __forceinline__ void step(T* v, int lane) {
    if constexpr (S < LOG) {
      constexpr int h = P >> (S + 1);
      const bool hi = (lane >> bit(S)) & 1;
#pragma unroll
      for (int j = 0; j < h; ++j) {
        const T a = v[j], b = v[j + h];
        v[j] = (hi ? b : a) + across<S>(hi ? a : b);
      }
      step<S + 1>(v, lane);
    } else if constexpr (S < 6) {
      v[0] += across<S>(v[0]);
      step<S + 1>(v, lane);
    }
  }
  // v: P values (0 beyond M)
  static __device__ __forceinline__ T run(T* v, int lane) {
    step<0>(v, lane);
    return v[0];
  }
  static __device__ __forceinline__ int index(int lane) {
    int r = 0;
#pragma unroll
    for (int s = 0; s < LOG; ++s) r |= ((lane >> bit(s)) & 1) << (LOG - 1 - s);
    return r;
  }
  // one lane of those that hold value index(l)
  static __device__ __forceinline__ bool holds(int lane) {
    int other = 0;
#pragma unroll
    for (int s = LOG; s < 6; ++s) other |= (lane >> bit(s)) & 1;
    return other == 0;
  }
};

}  // namespace garfield

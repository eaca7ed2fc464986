// Where the streaming kernels find the n vectors they read: the rows of one
// row-major n x d matrix, or a table of row pointers -- one segment of n
// vectors stored apart (the same layer's gradient from each of n workers, or
// n whole vectors in separate buffers).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace garfield {

struct MatrixRows {
  const float* x;
  int64_t d;
  __device__ __forceinline__ const float* row(int64_t i) const { return x + i * d; }
};

struct TableRows {
  const float* const* p;  // p[i] = vector i's segment
  __device__ __forceinline__ const float* row(int64_t i) const { return p[i]; }
};

// A batch of segments for one launch, passed by value in the kernel
// arguments: each segment's length, its first workgroup, and the coordinates
// one of its workgroups covers (distances) or its output (the aggregation
// kernels, whose workgroups all cover the same). Workgroup b works on the
// segment s with first[s] <= b < first[s + 1]. As many segments as the 4 KB of
// kernel arguments hold: every launch ends with a tail of its own (161 layers
// of 11.2 M coordinates in all, n = 11: 181 us a step in one launch per
// pass, 190 in two).
constexpr int kSegMax = 192;
struct SegTable {
  int count;
  int32_t first[kSegMax + 1];  // first[count] = workgroups of the launch
  int64_t dims[kSegMax];
  union {
    int64_t span[kSegMax];
    float* outs[kSegMax];
  };
};
static_assert(sizeof(SegTable) <= 3968, "room for the other arguments in 4 KB");

// The segment of workgroup b: the largest s with first[s] <= b (empty segments
// share their start with the next one and are skipped).
__device__ __forceinline__ int seg_of(const SegTable& t, int b) {
  int lo = 0, hi = t.count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (t.first[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

}  // namespace garfield

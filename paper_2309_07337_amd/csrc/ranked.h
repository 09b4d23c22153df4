// Device helpers for arrays whose elements belong to ranks in order (rank r's
// are [starts[r], starts[r + 1])): finding an element's rank, and walking such
// an array.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace hx {

constexpr int kWalkThreads = 256;
constexpr int kWalkChunk = 2048;  // consecutive elements a workgroup takes at a time

// Largest p in [0, R) with starts[p] <= v.
__device__ __forceinline__ int upper_rank(const int64_t* __restrict__ starts, int R, int64_t v) {
  int lo = 0, hi = R - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (starts[mid] <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The same from a rank r with starts[r] <= v: usually r itself or one of the
// next few, else a search of the ranks after them.
__device__ __forceinline__ int seek_rank(const int64_t* __restrict__ starts, int R, int r, int64_t v) {
#pragma unroll 1
  for (int k = 0; k < 4; ++k) {
    if (r + 1 >= R || starts[r + 1] > v) return r;
    ++r;
  }
  int lo = r, hi = R - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (starts[mid] <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The same for arbitrary v in [0, starts[R]): the rank that evenly divided
// starts would give, or a neighbour, else a search.
__device__ __forceinline__ int guess_rank(const int64_t* __restrict__ starts, int R, int64_t v) {
  const int64_t n = starts[R];
  int g = (int)((float)v * ((float)R / (float)n));
  g = max(0, min(g, R - 1));
  if (starts[g] <= v) {
    if (starts[g + 1] > v) return g;
    if (g + 2 <= R && starts[g + 2] > v) return g + 1;
  } else if (g > 0 && starts[g - 1] <= v) {
    return g - 1;
  }
  return upper_rank(starts, R, v);
}

// Calls f(i, rank) for i in [0, n), a chunk of consecutive elements per
// workgroup of kWalkThreads.  One search per chunk, then each lane's rank only
// moves on; in a chunk of one rank (most, where ranks have more elements than a
// chunk) nothing is looked up, and the lane's elements are in flight together.
// A search per element was a serial chain of ten loads on 1024 ranks: 78 us a
// pass over 8.4 M entries, 25 so.
template <class F>
__device__ __forceinline__ void for_ranked(int64_t n, const int64_t* __restrict__ starts, int R, F f) {
  constexpr int kItems = kWalkChunk / kWalkThreads;
  for (int64_t c0 = (int64_t)blockIdx.x * kWalkChunk; c0 < n; c0 += (int64_t)gridDim.x * kWalkChunk) {
    const int64_t c1 = min(c0 + (int64_t)kWalkChunk, n);
    int r = upper_rank(starts, R, c0);
    if (c0 + kWalkChunk <= n && (r + 1 >= R || starts[r + 1] >= c1)) {
#pragma unroll
      for (int k = 0; k < kItems; ++k) f(c0 + threadIdx.x + k * kWalkThreads, r);
      continue;
    }
    for (int64_t i = c0 + threadIdx.x; i < c1; i += kWalkThreads) {
      r = seek_rank(starts, R, r, i);
      f(i, r);
    }
  }
}

inline unsigned walk_blocks(int64_t n) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + kWalkChunk - 1) / kWalkChunk, 1 << 16));
}

}  // namespace hx

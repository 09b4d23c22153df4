// Plans of a persistent neighborhood all-to-all-v, built on the GPU for every
// rank of a decomposition (all setup at initialisation, MPI Advance Sec. 2.2).
//
// Data structures (no sorting anywhere; order comes from bit positions and
// prefix sums):
//   B[r]      bitmap over global columns of rank r's off-rank references
//             (halo discovery; compacting it with a block-wide prefix scan of
//             popcounts yields the halo N_r sorted and duplicate-free)
//   M[r][q]   |N_r ∩ owned(q)|: dense rank-pair message sizes.  Its rows are
//             the receive lists; its transpose gives the send lists; row
//             prefix sums give every displacement
//   NB[m]     node bitmap: OR of B[s] over the ranks s of node m.  A set bit c
//             owned by a remote rank q is one entry of the deduplicated
//             aggregated message D(q -> m) (a value crosses a node pair once,
//             Sec. 2.2, last paragraph); its position inside D(q -> m) is a
//             bitmap rank (popcount prefix)
// Every list entry is then written by a scatter whose destination is a closed
// form of these prefix sums, so the result is deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <memory>
#include <numeric>
#include <vector>

#include "common.h"
#include "internal.h"
#include "ranked.h"

namespace hx {
namespace {

constexpr int TB = kWalkThreads;

unsigned blocks_for(int64_t n, int per = TB) {
  int64_t b = (n + per - 1) / per;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 1 << 16));
}

#define GRID_STRIDE(i, n) \
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// Placement of R ranks on NN = ceil(R / ppn) nodes (Sec. 2.2 groups ranks by
// node without fixing which ranks share one).  Block: node p / ppn, local rank
// p % ppn, the last node may hold fewer ranks.  Cyclic (round robin): node
// p % NN, local rank p / NN.
struct Place {
  int R, ppn, NN, cyc;
  __device__ int node(int p) const { return cyc ? p % NN : p / ppn; }
  __device__ int lrank(int p) const { return cyc ? p / NN : p % ppn; }
  __device__ int cnt(int m) const { return cyc ? (R - 1 - m) / NN + 1 : min(ppn, R - m * ppn); }
  __device__ int rank_at(int m, int l) const { return cyc ? l * NN + m : m * ppn + l; }
  // The rank of node m that receives rank q's deduplicated message: the one
  // whose local rank is q's modulo the size of node m.
  __device__ int partner(int q, int m) const { return rank_at(m, lrank(q) % cnt(m)); }
};

// 3-step (one message per node pair, block placement only): the rank of node
// n that sends node n's data for node m, and the rank of node m that receives it.
__device__ __forceinline__ int aggr_of(const Place& P, int n, int m) { return P.rank_at(n, m % P.cnt(n)); }
__device__ __forceinline__ int recv_of(const Place& P, int n, int m) { return P.rank_at(m, n % P.cnt(m)); }
// The forwarder on node m of the entries owned by rank q (the rank their
// aggregated stage-1 message lands on), the sender of that message, and the
// first row of the column range the message deduplicates over.
__device__ __forceinline__ int fwd_of(const Place& P, int q, int m, int v3) {
  return v3 ? recv_of(P, P.node(q), m) : P.partner(q, m);
}
__device__ __forceinline__ int agg_sender(const Place& P, int q, int m, int v3) {
  return v3 ? aggr_of(P, P.node(q), m) : q;
}
__device__ __forceinline__ int64_t agg_base(const Place& P, int q, const int64_t* __restrict__ rs, int v3) {
  return v3 ? rs[P.rank_at(P.node(q), 0)] : rs[q];
}

template <class T>
__device__ T wave_sum(T v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Block-wide sum (every thread gets it).  blockDim.x is a multiple of 64, <= 1024.
template <class T>
__device__ T block_sum(T v) {
  __shared__ T sh[16];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  v = wave_sum(v);
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  T t = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
  __syncthreads();
  return t;
}

// Block-wide exclusive scan; *total = block sum.
template <class T>
__device__ T block_exscan(T v, T* total) {
  __shared__ T sh[16];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  T x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  T base = 0, tot = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
    if (i < wid) base += sh[i];
    tot += sh[i];
  }
  __syncthreads();
  *total = tot;
  return base + x - v;
}

// Rank of bit c in bitmap row (words NB, exclusive word prefix NBP): number of
// set bits below c.  Rows carry one extra zero word so c may equal n.
__device__ __forceinline__ int32_t bit_rank(const uint32_t* __restrict__ NB, const int32_t* __restrict__ NBP,
                                            int64_t c) {
  const int64_t w = c >> 5;
  const uint32_t below = (uint32_t)((1ull << (c & 31)) - 1ull);
  return NBP[w] + __popc(NB[w] & below);
}

// ---------------------------------------------------------------------------
// Generic device utilities
// ---------------------------------------------------------------------------
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_BLOCK = TB * SCAN_ITEMS;

// POPC: the scan of the words' popcounts instead of the values themselves.
template <bool POPC>
__device__ __forceinline__ int32_t scan_value(const int32_t* __restrict__ in, int64_t i) {
  return POPC ? __popc((uint32_t)in[i]) : in[i];
}

template <bool POPC>
__global__ void k_scan_partials(const int32_t* __restrict__ in, int64_t n, int64_t* __restrict__ part) {
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK;
  int64_t s = 0;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    const int64_t i = base + (int64_t)k * TB + threadIdx.x;
    if (i < n) s += scan_value<POPC>(in, i);
  }
  s = block_sum(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void k_scan_part_scan(int64_t* part, int64_t nparts) {
  int64_t base = 0;
  for (int64_t c0 = 0; c0 < nparts; c0 += blockDim.x) {
    const int64_t i = c0 + threadIdx.x;
    const int64_t v = i < nparts ? part[i] : 0;
    int64_t tot;
    const int64_t pre = block_exscan(v, &tot);
    if (i < nparts) part[i] = base + pre;
    base += tot;
  }
  if (threadIdx.x == 0) part[nparts] = base;
}

template <bool POPC>
__global__ void k_scan_final(const int32_t* __restrict__ in, int64_t n, const int64_t* __restrict__ part,
                             int32_t* __restrict__ out) {
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK;
  // each thread takes SCAN_ITEMS consecutive items
  const int64_t i0 = base + (int64_t)threadIdx.x * SCAN_ITEMS;
  int64_t v[SCAN_ITEMS];
  int64_t s = 0;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    v[k] = (i0 + k < n) ? scan_value<POPC>(in, i0 + k) : 0;
    s += v[k];
  }
  int64_t tot;
  int64_t run = part[blockIdx.x] + block_exscan(s, &tot);
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    if (i0 + k < n) out[i0 + k] = (int32_t)run;
    run += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = (int32_t)part[gridDim.x];
}

// The scan's launches alone; part holds scan_parts(n) values.
int64_t scan_parts(int64_t n) { return std::max<int64_t>(1, (n + SCAN_BLOCK - 1) / SCAN_BLOCK) + 1; }
template <bool POPC = false>
int scan_launch(const int32_t* in, int32_t* out, int64_t n, int64_t* part, hipStream_t s) {
  const int64_t nb = scan_parts(n) - 1;
  hipLaunchKernelGGL(k_scan_partials<POPC>, dim3((unsigned)nb), dim3(TB), 0, s, in, n, part);
  HX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_scan_part_scan, dim3(1), dim3(1024), 0, s, part, nb);
  HX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_scan_final<POPC>, dim3((unsigned)nb), dim3(TB), 0, s, in, n, part, out);
  HX_HIP(hipGetLastError());
  return HX_SUCCESS;
}

// Grouping entries by key is a stable radix sort of (key, entry): groups come
// out in key order with their entries ascending, whatever the distribution of
// the keys (no atomics on memory, no per-group sort; a key that every entry
// shares costs what any other does).  Per digit a histogram pass, a scan of
// the (digit, block) table and a scatter pass.  A block sorts its 4096 pairs
// by digit in LDS first, so that its scattered writes are runs of whole lines:
// 4-byte writes straight to their places cost a memory sector each (220 us a
// pass for 10 M pairs, 10-bit digits), and digits of more than 8 bits would
// leave runs shorter than a line.  Counting and placing with atomics and an
// insertion sort per group took 843 us for 10 M entries over 2^20 keys, this
// 260 us (histograms 49, scans 39, scatters 157, pointers 15).
constexpr int RS_WAVES = TB / 64;
constexpr int RS_STEPS = 16;                              // pairs per lane
constexpr int RS_BLOCK = RS_WAVES * 64 * RS_STEPS;        // pairs per workgroup
constexpr int RS_MAX_BITS = 8;
static_assert((1 << RS_MAX_BITS) == TB, "one thread per digit");

// hist[digit * nblocks + block] = this block's entries with that digit.  With
// err (the first digit's pass) keys outside [0, nkeys) are reported.
__global__ void __launch_bounds__(TB) k_radix_hist(const int32_t* __restrict__ keys, int64_t n, int64_t nkeys,
                                                   int shift, int bits, int32_t* __restrict__ hist, int nblocks,
                                                   int* err) {
  __shared__ int32_t s_cnt[1 << RS_MAX_BITS];
  const int B = 1 << bits;
  s_cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * RS_BLOCK + threadIdx.x;
  bool bad = false;
#pragma unroll
  for (int k = 0; k < RS_STEPS; ++k) {
    const int64_t i = i0 + (int64_t)k * TB;
    if (i < n) {
      const int32_t key = keys[i];
      bad |= key < 0 || key >= nkeys;
      atomicAdd(&s_cnt[((uint32_t)key >> shift) & (B - 1)], 1);
    }
  }
  if (err != nullptr && bad) atomicOr(err, 16);
  __syncthreads();
  if ((int)threadIdx.x < B) hist[(size_t)threadIdx.x * nblocks + blockIdx.x] = s_cnt[threadIdx.x];
}

// Moves (key, value) pairs to their places in this digit's order; vals_in
// null: the values are the entry numbers.  Each wavefront takes a contiguous
// run of the block's pairs, 64 at a time: a lane's rank among the lanes of its
// digit comes from ballots, the run's next place per digit from LDS.
__global__ void __launch_bounds__(TB) k_radix_scatter(const int32_t* __restrict__ keys_in,
                                                      const int32_t* __restrict__ vals_in, int64_t n, int shift,
                                                      int bits, const int32_t* __restrict__ offs, int nblocks,
                                                      int32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out) {
  __shared__ int32_t s_next[RS_WAVES][1 << RS_MAX_BITS];
  __shared__ int32_t s_dst[1 << RS_MAX_BITS];  // place in the output less place in the block, per digit
  __shared__ int32_t s_key[RS_BLOCK], s_val[RS_BLOCK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
  for (int w = 0; w < RS_WAVES; ++w) s_next[w][tid] = 0;
  __syncthreads();
  const int64_t b0 = (int64_t)blockIdx.x * RS_BLOCK;
  const int64_t i0 = b0 + wave * (64 * RS_STEPS) + lane;
  int32_t key[RS_STEPS], val[RS_STEPS];
#pragma unroll
  for (int k = 0; k < RS_STEPS; ++k) {
    const int64_t i = i0 + k * 64;
    key[k] = i < n ? keys_in[i] : 0;
    val[k] = vals_in == nullptr ? (int32_t)i : (i < n ? vals_in[i] : 0);
  }
#pragma unroll
  for (int k = 0; k < RS_STEPS; ++k)
    if (i0 + k * 64 < n) atomicAdd(&s_next[wave][((uint32_t)key[k] >> shift) & mask], 1);
  __syncthreads();
  {  // counts -> first places in the block, one thread per digit
    int32_t c[RS_WAVES], sum = 0, tot;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) sum += (c[w] = s_next[w][tid]);
    int32_t at = block_exscan(sum, &tot);
    if (tid <= (int)mask) s_dst[tid] = offs[(size_t)tid * nblocks + blockIdx.x] - at;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) {
      s_next[w][tid] = at;
      at += c[w];
    }
  }
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int k = 0; k < RS_STEPS; ++k) {
    const bool in = i0 + k * 64 < n;
    const uint32_t d = ((uint32_t)key[k] >> shift) & mask;
    uint64_t same = __ballot(in);
    for (int b = 0; b < bits; ++b) {
      const bool one = (d >> b) & 1u;
      const uint64_t v = __ballot(one);
      same &= one ? v : ~v;
    }
    if (in) {
      const int32_t at = s_next[wave][d] + __popcll(same & below);
      s_key[at] = key[k];
      s_val[at] = val[k];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (in && (same & below) == 0) s_next[wave][d] += __popcll(same);  // the digit's first lane
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  __syncthreads();
  const int cnt = (int)min((int64_t)RS_BLOCK, n - b0);
  for (int j = tid; j < cnt; j += TB) {
    const int32_t kj = s_key[j];
    const int32_t at = s_dst[((uint32_t)kj >> shift) & mask] + j;
    keys_out[at] = kj;
    vals_out[at] = s_val[j];
  }
}

// ptr[k] = first sorted entry with key >= k, for k in [0, nkeys].  Entry i
// gives the keys after its predecessor's up to its own; runs of more than a
// few keys without entries are filled by a wavefront each, the keys before
// the first and after the last entry by the whole grid.  Writes nothing where a
// key was found outside [0, nkeys) (err set): such a key is no place in ptr.
constexpr int CHUNK = 2048;  // consecutive items a block takes at a time
__global__ void __launch_bounds__(TB) k_group_ptr(const int32_t* __restrict__ skeys, int64_t n, int64_t nkeys,
                                                  int32_t* __restrict__ ptr, const int* __restrict__ err) {
  __shared__ int32_t s_entry[CHUNK], s_from[CHUNK], s_to[CHUNK];  // runs to fill: keys (from, to]
  __shared__ int s_gaps;
  if (err != nullptr && *err != 0) return;  // (uniform)
  const int64_t first = n > 0 ? min((int64_t)skeys[0], nkeys) : nkeys;
  const int64_t last = n > 0 ? min((int64_t)skeys[n - 1], nkeys) : nkeys;
  const int64_t gid = (int64_t)blockIdx.x * TB + threadIdx.x, gsz = (int64_t)gridDim.x * TB;
  for (int64_t k = gid; k <= first; k += gsz) ptr[k] = 0;
  for (int64_t k = last + 1 + gid; k <= nkeys; k += gsz) ptr[k] = (int32_t)n;
  for (int64_t c0 = (int64_t)blockIdx.x * CHUNK; c0 < n; c0 += (int64_t)gridDim.x * CHUNK) {
    if (threadIdx.x == 0) s_gaps = 0;
    __syncthreads();
    const int64_t c1 = min(c0 + CHUNK, n);
    for (int64_t i = c0 + threadIdx.x; i < c1; i += TB) {
      if (i == 0) continue;
      const int64_t a = skeys[i - 1], b = min((int64_t)skeys[i], nkeys);
      if (b - a <= 8) {
        for (int64_t k = a + 1; k <= b; ++k) ptr[k] = (int32_t)i;
      } else {
        const int g = atomicAdd(&s_gaps, 1);
        s_entry[g] = (int32_t)i;
        s_from[g] = (int32_t)a;
        s_to[g] = (int32_t)b;
      }
    }
    __syncthreads();
    for (int g = threadIdx.x >> 6; g < s_gaps; g += RS_WAVES) {
      const int64_t b = s_to[g];
      for (int64_t k = (int64_t)s_from[g] + 1 + (threadIdx.x & 63); k <= b; k += 64) ptr[k] = s_entry[g];
    }
    __syncthreads();  // the gap list is reused
  }
}

// err |= 16 if some idx[i] is outside [0, hi).
__global__ void k_check_range(const int32_t* __restrict__ idx, int64_t n, int64_t hi, int* err) {
  GRID_STRIDE(i, n) {
    const int32_t v = idx[i];
    if (v < 0 || v >= hi) atomicOr(err, 16);
  }
}

__global__ void k_flag(const int32_t* __restrict__ idx, int64_t n, int64_t domain, unsigned char* flags) {
  GRID_STRIDE(i, n) {
    const int32_t v = idx[i];
    if (v >= 0 && v < domain) flags[v] = 1;
  }
}

// *out += number of set flags (nwords words of four).  One atomic a block, so
// few blocks: 4096 blocks adding to one address took 420 us for 1 M flags.
__global__ void k_count_flags(const uint32_t* __restrict__ flags, int64_t nwords, unsigned long long* out) {
  int64_t s = 0;
  GRID_STRIDE(i, nwords) s += __popc(flags[i]);
  s = block_sum(s);
  if (threadIdx.x == 0) atomicAdd(out, (unsigned long long)s);
}

// *out += number of segments of a CSR that are not empty.
__global__ void k_count_nonempty(const int32_t* __restrict__ ptr, int64_t n, unsigned long long* out) {
  int64_t s = 0;
  GRID_STRIDE(i, n) s += ptr[i + 1] > ptr[i] ? 1 : 0;
  s = block_sum(s);
  if (threadIdx.x == 0) atomicAdd(out, (unsigned long long)s);
}

// ---------------------------------------------------------------------------
// Halo discovery
// ---------------------------------------------------------------------------
// Checks the row pointers of rows [i0, i0 + rows) (err |= 8 where they
// decrease) and notes where the entries of ranks r0, r0 + 1, ... r0 + g - 1
// start and end.
__global__ void k_rank_entries(const int64_t* __restrict__ rs, int64_t i0, int64_t rows, int r0, int g,
                               const int64_t* __restrict__ row_ptr, int64_t* __restrict__ ent, int* err) {
  bool bad = false;
  GRID_STRIDE(k, rows) bad |= row_ptr[i0 + k + 1] < row_ptr[i0 + k];
  if (bad) atomicOr(err, 8);
  GRID_STRIDE(r, (int64_t)g + 1) ent[r] = row_ptr[rs[r0 + r]];
}

// Marks the off-rank columns of the entries of ranks r0 .. r0 + g - 1 in their
// ranks' bitmaps (rows of Wp words of B, counted from r0).  Entry-parallel: a
// workgroup streams chunks of consecutive entries, whose rank rarely changes
// within a chunk.  Bound by the stream of columns and the atomics of the
// off-rank ones; a bit that is seen set already needs none (a 27-point rank
// names a halo column nine times).  A lane walking its own row read 27 columns
// at a stride of 108 bytes instead: 899 us for the 56.6 M entries of 512
// ranks; 171 us so.  (33.6 M random entries of 1024 ranks, 10 M of them marks
// all over 134 MB: 441 and 455 us.)
// Writes nothing where the row pointers were found to decrease (their range
// is then not known to be the columns').
constexpr int kMarkItems = 16;
// (bitmap rows are whole 16-byte vectors)
__device__ __forceinline__ int popc4(const uint4 v) { return __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w); }
__global__ void __launch_bounds__(TB) k_mark_csr(const int64_t* __restrict__ rs, int64_t n, int r0, int g,
                                                 const int64_t* __restrict__ ent, const int32_t* __restrict__ cols,
                                                 uint32_t* B, int64_t Wp, int* err) {
  if (*(volatile int*)err & 8) return;
  const int64_t end = ent[g], step = (int64_t)gridDim.x * (TB * kMarkItems);
  bool bad = false;
  for (int64_t c0 = ent[0] + (int64_t)blockIdx.x * (TB * kMarkItems); c0 < end; c0 += step) {
    int32_t c[kMarkItems];
#pragma unroll
    for (int k = 0; k < kMarkItems; ++k) {
      const int64_t e = c0 + threadIdx.x + k * TB;
      c[k] = e < end ? __builtin_nontemporal_load(cols + e) : 0;
    }
    int r = upper_rank(ent, g, c0);
    int64_t lo = rs[r0 + r], hi = rs[r0 + r + 1], next = ent[r + 1];
#pragma unroll
    for (int k = 0; k < kMarkItems; ++k) {
      const int64_t e = c0 + threadIdx.x + k * TB;
      if (e >= end) break;
      if (e >= next) {
        r = seek_rank(ent, g, r, e);
        lo = rs[r0 + r], hi = rs[r0 + r + 1], next = ent[r + 1];
      }
      if (c[k] < 0 || c[k] >= n) bad = true;
      else if (c[k] < lo || c[k] >= hi) {
        uint32_t* w = B + (size_t)r * Wp + (c[k] >> 5);
        const uint32_t bit = 1u << (c[k] & 31);
        if ((*w & bit) == 0) atomicOr(w, bit);
      }
    }
  }
  if (bad) atomicOr(err, 1);
}

// The same with the bitmap of one rank and 2^kMarkSegBits columns in LDS: a
// workgroup streams its rank's entries once, then writes the segment's words
// whole (nothing is cleared beforehand) and counts them.  Workgroups of one
// rank are dispatched one after the other on one XCD, whose L2 then serves
// the later streams.  171 -> 109 us and 455 -> 63 us for the matrices above,
// without the clearing and counting passes (25 + 21 us).
constexpr int kMarkSegBits = 20;  // 128 KiB
constexpr int kMarkThreads = 1024;
constexpr int kMarkMaxSegs = 4;   // streams of the entries at most
constexpr int kMarkMinRanks = 8;  // workgroups at least, below which the chip is idle
__global__ void __launch_bounds__(kMarkThreads) k_mark_lds(const int64_t* __restrict__ rs, int64_t n, int r0, int g,
                                                           int nseg, const int64_t* __restrict__ ent,
                                                           const int32_t* __restrict__ cols, uint32_t* __restrict__ B,
                                                           int64_t Wp, unsigned long long* cnt, int* err) {
  extern __shared__ __align__(16) uint32_t s_bits[];
  const int r = (int)(blockIdx.x / (8 * nseg)) * 8 + (int)(blockIdx.x & 7), seg = (int)(blockIdx.x >> 3) % nseg;
  if (r >= g || (*(volatile int*)err & 8)) return;
  const int64_t w0 = (int64_t)seg << (kMarkSegBits - 5);
  const int nv = (int)(min((int64_t)1 << (kMarkSegBits - 5), Wp - w0) / 4);  // 16-byte vectors of the segment
  uint4* s_vec = reinterpret_cast<uint4*>(s_bits);
  for (int i = threadIdx.x; i < nv; i += kMarkThreads) s_vec[i] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  const int64_t c0 = (int64_t)seg << kMarkSegBits, lo = rs[r0 + r], hi = rs[r0 + r + 1], e1 = ent[r + 1];
  bool bad = false;
  for (int64_t e0 = ent[r] + threadIdx.x; e0 < e1; e0 += kMarkThreads * kMarkItems) {
    int32_t c[kMarkItems];
#pragma unroll
    for (int k = 0; k < kMarkItems; ++k) {
      const int64_t e = e0 + k * kMarkThreads;
      c[k] = e < e1 ? cols[e] : (int32_t)lo;  // (an own column is left out)
    }
#pragma unroll
    for (int k = 0; k < kMarkItems; ++k) {
      const bool in = c[k] >= 0 && c[k] < n, own = c[k] >= lo && c[k] < hi;
      bad |= !in && e0 + k * kMarkThreads < e1;
      const int64_t o = c[k] - c0;
      if (in && !own && (uint64_t)o >> kMarkSegBits == 0) atomicOr(&s_bits[o >> 5], 1u << (o & 31));
    }
  }
  if (bad) atomicOr(err, 1);
  __syncthreads();
  int total = 0;
  uint4* out = reinterpret_cast<uint4*>(B + (size_t)r * Wp + w0);
  for (int i = threadIdx.x; i < nv; i += kMarkThreads) {
    const uint4 v = s_vec[i];
    total += popc4(v);
    out[i] = v;
  }
  const int64_t t = block_sum((int64_t)total);
  if (threadIdx.x == 0 && t) atomicAdd(cnt + r, (unsigned long long)t);
}

// Bitmap rows are read by workgroups of kBitThreads.
constexpr int kBitThreads = 1024;

// Number of set bits of each rank's bitmap (one block per rank).
__global__ void __launch_bounds__(kBitThreads) k_popc_rows(const uint32_t* __restrict__ B, int64_t Wp, int64_t* cnt) {
  const uint4* __restrict__ Br = reinterpret_cast<const uint4*>(B + (size_t)blockIdx.x * Wp);
  const int64_t nv = Wp / 4;
  int s = 0;
#pragma unroll 4
  for (int64_t w = threadIdx.x; w < nv; w += kBitThreads) s += popc4(Br[w]);
  const int64_t t = block_sum((int64_t)s);
  if (threadIdx.x == 0) cnt[blockIdx.x] = t;
}

// Writes the set bits of each rank's bitmap as ascending column ids.
__global__ void __launch_bounds__(kBitThreads) k_compact_bits(const uint32_t* __restrict__ B, int64_t Wp,
                                                              const int64_t* __restrict__ off,
                                                              int32_t* __restrict__ out) {
  const uint4* __restrict__ Br = reinterpret_cast<const uint4*>(B + (size_t)blockIdx.x * Wp);
  const int64_t end = off[blockIdx.x + 1], nv = Wp / 4;
  int64_t base = off[blockIdx.x];
  const uint4 none = make_uint4(0, 0, 0, 0);
  uint4 next = threadIdx.x < nv ? Br[threadIdx.x] : none;
  for (int64_t w0 = 0; w0 < nv; w0 += kBitThreads) {
    const uint4 v = next;
    const int64_t w = w0 + threadIdx.x, wn = w + kBitThreads;
    next = wn < nv ? Br[wn] : none;  // in flight during this round's scan
    int tot;
    int64_t o = base + block_exscan(popc4(v), &tot);
    const uint32_t words[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t bits = words[k];
      while (bits) {
        const int b = __ffs(bits) - 1;
        if (o < end) out[o] = (int32_t)((w * 4 + k) * 32 + b);
        ++o;
        bits &= bits - 1u;
      }
    }
    base += tot;
  }
}

// Per halo entry: its rank, its owner, and the rank-pair count M[r][q].  A
// rank's halo is sorted, so the entries of a pair are one run: its first entry
// subtracts its position, its last adds the next one (two atomics a pair that
// do not meet, instead of one an entry that mostly do).  8.3 M entries of 1024
// ranks: 436 -> 77 us.
__global__ void k_entry_info(const int32_t* __restrict__ hcol, int64_t nH, const int64_t* __restrict__ hoff,
                             const int64_t* __restrict__ rs, int R, int64_t n, int check, int32_t* hrank,
                             int32_t* own, int32_t* M, int* err) {
  for_ranked(nH, hoff, R, [&](int64_t e, int r) {
    const int64_t c = hcol[e];
    const bool first = e == hoff[r], last = e + 1 == hoff[r + 1];
    const int64_t before = first ? -1 : hcol[e - 1], after = last ? n : hcol[e + 1];
    if (check) {
      if (c < 0 || c >= n) {
        atomicOr(err, 1);
        return;
      }
      if (before >= c) atomicOr(err, 2);
      if (c >= rs[r] && c < rs[r + 1]) {
        atomicOr(err, 4);
        return;
      }
    }
    const int q = guess_rank(rs, R, c);
    hrank[e] = r;
    own[e] = q;
    int32_t* m = M + (size_t)r * R + q;
    const bool starts = first || before < rs[q], ends = last || after >= rs[q + 1];
    if (starts && ends) atomicAdd(m, 1);
    else if (starts) atomicAdd(m, -(int32_t)e);
    else if (ends) atomicAdd(m, (int32_t)(e + 1));
  });
}

// ---------------------------------------------------------------------------
// Dense rank-pair tables
// ---------------------------------------------------------------------------
__global__ void k_transpose(const int32_t* __restrict__ A, int32_t* __restrict__ AT, int R) {
  __shared__ int32_t t[32][33];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  for (int y = threadIdx.y; y < 32; y += blockDim.y) {
    const int r = by + y, c = bx + threadIdx.x;
    if (r < R && c < R) t[y][threadIdx.x] = A[(size_t)r * R + c];
  }
  __syncthreads();
  for (int y = threadIdx.y; y < 32; y += blockDim.y) {
    const int r = bx + y, c = by + threadIdx.x;
    if (r < R && c < R) AT[(size_t)r * R + c] = t[threadIdx.x][y];
  }
}

// Row-wise exclusive prefix P, row sums and row nonzero counts (block per row).
__global__ void k_row_exscan(const int32_t* __restrict__ A, int32_t* __restrict__ P, int R, int64_t* rowsum,
                             int64_t* rownnz) {
  const size_t r = blockIdx.x;
  int64_t base = 0, nnz = 0;
  for (int c0 = 0; c0 < R; c0 += blockDim.x) {
    const int c = c0 + threadIdx.x;
    const int32_t v = c < R ? A[r * R + c] : 0;
    int64_t tot;
    const int64_t pre = block_exscan((int64_t)v, &tot);
    if (c < R) P[r * R + c] = (int32_t)(base + pre);
    base += tot;
    nnz += block_sum((int64_t)(v != 0));
  }
  if (threadIdx.x == 0) {
    rowsum[r] = base;
    rownnz[r] = nnz;
  }
}

// Nonzeros of each row as (column, value, prefix) lists (block per row).
__global__ void k_row_compact(const int32_t* __restrict__ A, const int32_t* __restrict__ P, int R,
                              const int64_t* __restrict__ list_off, int32_t* procs, int32_t* counts,
                              int32_t* displs) {
  const size_t r = blockIdx.x;
  const int64_t end = list_off[r + 1];
  int64_t base = list_off[r];
  for (int c0 = 0; c0 < R; c0 += blockDim.x) {
    const int c = c0 + threadIdx.x;
    const int32_t v = c < R ? A[r * R + c] : 0;
    int64_t tot;
    const int64_t pre = block_exscan((int64_t)(v != 0), &tot);
    if (v != 0 && base + pre < end) {
      const int64_t o = base + pre;
      procs[o] = c;
      counts[o] = v;
      displs[o] = P[r * R + c];
    }
    base += tot;
  }
}

// ---------------------------------------------------------------------------
// Locality-aware (2-step) tables
// ---------------------------------------------------------------------------
// NB: one workgroup per node and segment of 2^seg_bits columns gathers the
// segment's bits in LDS from the sorted halos of the node's ranks and writes
// its words whole (no clearing, no atomics on memory).  8.3 M entries on 32
// nodes: 139 -> 25 us.
constexpr int kSegBitsMin = 13, kSegBitsMax = 19;  // 1 to 64 KiB of LDS
__device__ __forceinline__ int64_t lower_entry(const int32_t* __restrict__ v, int64_t lo, int64_t hi, int64_t x) {
  while (lo < hi) {  // first entry with v >= x
    const int64_t mid = (lo + hi) >> 1;
    if (v[mid] < x) lo = mid + 1; else hi = mid;
  }
  return lo;
}
__global__ void __launch_bounds__(512) k_node_mark(const int32_t* __restrict__ hcol, const int64_t* __restrict__ hoff,
                                                   Place P, int seg_bits, uint32_t* __restrict__ NB, int64_t W1) {
  extern __shared__ uint32_t s_bits[];
  const int nseg = gridDim.x / P.NN;
  const int m = blockIdx.x / nseg;
  const int64_t c0 = (int64_t)(blockIdx.x % nseg) << seg_bits, c1 = c0 + ((int64_t)1 << seg_bits);
  const int nw = 1 << (seg_bits - 5);
  for (int i = threadIdx.x; i < nw; i += blockDim.x) s_bits[i] = 0;
  __syncthreads();
  // the ranges of up to 256 ranks at a time (one search a lane), then a
  // wavefront per rank
  __shared__ int64_t s_at[512];
  const int cnt = P.cnt(m), waves = blockDim.x >> 6, lane = threadIdx.x & 63;
  for (int l0 = 0; l0 < cnt; l0 += 256) {
    const int l = l0 + (threadIdx.x >> 1);
    __syncthreads();
    if (l < cnt) {
      const int r = P.rank_at(m, l);
      s_at[threadIdx.x] = lower_entry(hcol, hoff[r], hoff[r + 1], (threadIdx.x & 1) ? c1 : c0);
    }
    __syncthreads();
    for (int k = threadIdx.x >> 6; k < min(256, cnt - l0); k += waves)
      for (int64_t e = s_at[2 * k] + lane; e < s_at[2 * k + 1]; e += 64) {
        const int32_t c = (int32_t)(hcol[e] - c0);
        atomicOr(&s_bits[c >> 5], 1u << (c & 31));
      }
  }
  __syncthreads();
  const int64_t w0 = c0 >> 5;
  for (int i = threadIdx.x; i < nw; i += blockDim.x)
    if (w0 + i < W1) NB[(size_t)m * W1 + w0 + i] = s_bits[i];
}

// MD[m][q] = |D(q -> m)| for q off node m (else 0).  3-step: |D(n -> m)| of
// q's node n at q = the pair's aggregator (else 0).
__global__ void k_dedup_counts(const uint32_t* __restrict__ NB, const int32_t* __restrict__ NBP, int64_t W1,
                               const int64_t* __restrict__ rs, Place P, int v3, int32_t* MD) {
  const int R = P.R;
  GRID_STRIDE(i, (int64_t)P.NN * R) {
    const int m = (int)(i / R), q = (int)(i % R);
    int32_t v = 0;
    if (P.node(q) != m) {
      const uint32_t* nb = NB + (size_t)m * W1;
      const int32_t* np = NBP + (size_t)m * W1;
      if (!v3) {
        v = bit_rank(nb, np, rs[q + 1]) - bit_rank(nb, np, rs[q]);
      } else {
        const int n = P.node(q);
        const int first = P.rank_at(n, 0);  // block: node n's rows are contiguous
        if (q == aggr_of(P, n, m))
          v = bit_rank(nb, np, rs[first + P.cnt(n)]) - bit_rank(nb, np, rs[first]);
      }
    }
    MD[i] = v;
  }
}

// Stage-1 message sizes S1[q][d]: direct to on-node d, deduplicated to partners.
__global__ void k_stage1_sizes(const int32_t* __restrict__ MT, const int32_t* __restrict__ MD, Place P, int v3,
                               int32_t* S1) {
  const int R = P.R;
  GRID_STRIDE(i, (int64_t)R * R) {
    const int q = (int)(i / R), d = (int)(i % R);
    int32_t v = 0;
    if (d != q) {
      const int nq = P.node(q), nd = P.node(d);
      if (nq == nd) v = MT[i];
      else if (v3 ? (q == aggr_of(P, nq, nd) && d == recv_of(P, nq, nd)) : d == P.partner(q, nd))
        v = MD[(size_t)nd * R + q];
    }
    S1[i] = v;
  }
}

// Stage-2 message sizes S2[t][s] (t forwards to s on its node): the entries of
// N_s owned by remote ranks whose aggregated message lands on t.
__global__ void k_stage2_sizes(const int32_t* __restrict__ M, Place P, int v3, int32_t* S2) {
  const int R = P.R;
  GRID_STRIDE(i, (int64_t)R * R) {
    const int t = (int)(i / R), s = (int)(i % R);
    int64_t v = 0;
    const int n = P.node(t);
    if (s != t && P.node(s) == n) {
      const int cn = P.cnt(n);
      const int lt = P.lrank(t);
      const int32_t* Ms = M + (size_t)s * R;
      for (int m = 0; m < P.NN; ++m) {
        if (m == n) continue;
        const int cm = P.cnt(m);
        if (v3) {  // every rank of the nodes whose pair message lands on t
          if (m % cn == lt)
            for (int l = 0; l < cm; ++l) v += Ms[P.rank_at(m, l)];
        } else {
          for (int l = lt; l < cm; l += cn) v += Ms[P.rank_at(m, l)];
        }
      }
    }
    S2[i] = (int32_t)v;
  }
}

// QP[s][q]: for q off s's node, the number of entries of N_s owned by the
// ranks before q (ascending) that share q's partner on s's node.  Class l0 of
// node n: the remote ranks whose local rank is l0 modulo the size of node n
// (3-step: every rank of the nodes m with m mod cn == l0).
__global__ void k_class_prefix(const int32_t* __restrict__ M, Place P, int v3, int32_t* QP) {
  const int R = P.R;
  GRID_STRIDE(i, (int64_t)R * P.ppn) {
    const int s = (int)(i / P.ppn), l0 = (int)(i % P.ppn);
    const int n = P.node(s);
    const int cn = P.cnt(n);
    if (l0 >= cn) continue;
    const int32_t* Ms = M + (size_t)s * R;
    int32_t* Qs = QP + (size_t)s * R;
    int32_t run = 0;
    if (P.cyc) {  // rank l*NN + m ascends with the local rank first, then the node
      for (int l = l0; l < P.ppn; l += cn)
        for (int m = 0; m < P.NN; ++m) {
          if (m == n || l >= P.cnt(m)) continue;
          const int q = P.rank_at(m, l);
          Qs[q] = run;
          run += Ms[q];
        }
      continue;
    }
    for (int m = 0; m < P.NN; ++m) {  // block: rank m*ppn + l ascends with the node first
      if (m == n) continue;
      const int cm = P.cnt(m);
      if (v3) {
        if (m % cn != l0) continue;
        for (int l = 0; l < cm; ++l) {
          const int q = P.rank_at(m, l);
          Qs[q] = run;
          run += Ms[q];
        }
      } else {
        for (int l = l0; l < cm; l += cn) {
          const int q = P.rank_at(m, l);
          Qs[q] = run;
          run += Ms[q];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// List entries (scatters with closed-form destinations)
// ---------------------------------------------------------------------------
// Stage-1 aggregated entries: one per set bit of a node bitmap owned off-node.
__global__ void k_s1_agg(const uint32_t* __restrict__ NB, const int32_t* __restrict__ NBP, int64_t W1,
                         int64_t W, const int64_t* __restrict__ rs, Place P, int v3,
                         const int32_t* __restrict__ PS1, const int64_t* __restrict__ s1_off, int32_t* s1_idx,
                         int* err) {
  const int R = P.R;
  GRID_STRIDE(i, (int64_t)P.NN * W) {
    const int m = (int)(i / W);
    const int64_t w = i % W;
    const uint32_t* nb = NB + (size_t)m * W1;
    const int32_t* np = NBP + (size_t)m * W1;
    uint32_t bits = nb[w];
    int q = -1;
    while (bits) {
      const int b = __ffs(bits) - 1;
      bits &= bits - 1u;
      const int64_t c = w * 32 + b;
      if (q < 0 || c >= rs[q + 1]) q = guess_rank(rs, R, c);  // (a word's columns mostly share their owner)
      if (P.node(q) == m) continue;
      const int t = fwd_of(P, q, m, v3);
      const int a = agg_sender(P, q, m, v3);
      const int64_t base = agg_base(P, q, rs, v3);
      const int64_t pos = s1_off[a] + PS1[(size_t)a * R + t] + (bit_rank(nb, np, c) - bit_rank(nb, np, base));
      if (pos < s1_off[a] || pos >= s1_off[a + 1]) {
        atomicOr(err, 32);
        continue;
      }
      s1_idx[pos] = (int32_t)(c - base);
    }
  }
}

// The list entries and the unpack slot of every halo entry (of rank s, owned by
// q), in one pass over the entries:
//   on the node, or a plain plan: a stage-1 send entry of q, unpacked from the
//     stage-1 slot of its message;
//   off the node, its aggregated message landing on s itself: unpacked from its
//     stage-1 slot there;
//   off the node, landing on another rank t of s's node: a stage-2
//     (redistribution) entry of t, unpacked from a stage-2 slot.
// 8.3 M entries of 1024 ranks, three passes 161 us, 107 so.
__global__ void k_entry_lists(const int32_t* __restrict__ hcol, const int32_t* __restrict__ hrank,
                              const int32_t* __restrict__ own, int64_t nH, const int64_t* __restrict__ hoff,
                              const int64_t* __restrict__ rs, Place P, int locality, int v3,
                              const int32_t* __restrict__ PS1, const int32_t* __restrict__ PS2,
                              const int32_t* __restrict__ QP, const int32_t* __restrict__ PM,
                              const int32_t* __restrict__ PR1, const int32_t* __restrict__ PR2,
                              const uint32_t* __restrict__ NB, const int32_t* __restrict__ NBP, int64_t W1,
                              const int64_t* __restrict__ s1_off, const int64_t* __restrict__ s2_off,
                              const int64_t* __restrict__ r1_tot, int32_t* __restrict__ s1_idx,
                              int32_t* __restrict__ s2_src, int32_t* __restrict__ unpack, int* err) {
  const int R = P.R;
  bool bad = false;
  GRID_STRIDE(e, nH) {
    const int s = hrank[e], q = own[e];
    const int64_t j = e - hoff[s], c = hcol[e];
    const size_t sq = (size_t)s * R + q;
    const int64_t in_msg = j - PM[sq];  // position among the entries of s owned by q
    const int n = locality ? P.node(s) : 0;
    if (!locality || P.node(q) == n) {
      const int64_t pos = s1_off[q] + PS1[(size_t)q * R + s] + in_msg;
      if (pos < s1_off[q] || pos >= s1_off[q + 1]) bad = true;
      else s1_idx[pos] = (int32_t)(c - agg_base(P, q, rs, v3));  // 3-step: rows of the node
      unpack[e] = (int32_t)(locality ? PR1[sq] + in_msg : j);
      continue;
    }
    const int t = fwd_of(P, q, n, v3);
    const uint32_t* nb = NB + (size_t)n * W1;
    const int32_t* np = NBP + (size_t)n * W1;
    const int32_t slot = PR1[(size_t)t * R + agg_sender(P, q, n, v3)] +
                         (bit_rank(nb, np, c) - bit_rank(nb, np, agg_base(P, q, rs, v3)));
    if (t == s) {
      unpack[e] = slot;
      continue;
    }
    const int64_t fwd = QP[sq] + in_msg;  // position in the message t forwards to s
    const int64_t pos = s2_off[t] + PS2[(size_t)t * R + s] + fwd;
    if (pos < s2_off[t] || pos >= s2_off[t + 1]) bad = true;
    else s2_src[pos] = slot;
    unpack[e] = (int32_t)(r1_tot[s] + PR2[(size_t)s * R + t] + fwd);
  }
  if (bad) atomicOr(err, 32);
}

// ---------------------------------------------------------------------------
// Transpose of the pack map
// ---------------------------------------------------------------------------
// Keys of the per-rank pack transposes: rank q's pack rows occupy
// [koff[q], koff[q+1]) of one key space (its own rows; its node's rows for
// the 3-step plan), so one stable grouping yields every rank's transpose.
__global__ void k_pack_keys(const int32_t* __restrict__ s1_idx, int64_t E, const int64_t* __restrict__ s1_off,
                            const int64_t* __restrict__ koff, int R, int32_t* keys, int* err) {
  bool bad = false;
  for_ranked(E, s1_off, R, [&](int64_t k, int q) {
    const int64_t key = koff[q] + s1_idx[k];
    bad |= key < koff[q] || key >= koff[q + 1];
    keys[k] = (int32_t)key;
  });
  if (bad) atomicOr(err, 16);
}

// A rank's transpose in LDS, one workgroup a rank: counts per row, their scan
// (the row pointers), then every slot placed under its row with atomics and the
// few slots of a row sorted.  Bound by the streams of slots in and out and the
// LDS atomics; the grouping by radix sort passes over keys and values three
// times and needs its keys and results rewritten per rank: 8.6 M slots of 1024
// ranks 311 -> 33 us, 0.9 M of 512 ranks 157 -> 18.
// (The slots of a row come nearly in order, so a lane's insertion sort is nearly
// one pass.)  Rows of more than kSortLane slots are sorted by the workgroup, as
// the set bits of a bitmap of the rank's slots (in the LDS that the slots leave:
// room of its own costs the workgroup beside it, 33 us -> 44).  The whole plan of 64 ranks of
// 20,000 rows, one of them packed for all ranks: 360 us (ranked one row after
// the other by the workgroup beyond 24 slots 2295, radix sort 479); of 64 ranks
// of 900 rows, each packed for 25 ranks: 325 (1556, 441); of 4096 ranks of 1024
// rows, one packed for all: 1579 (9833, 2328).
constexpr int kSortLane = 256;
constexpr int kTransMinRanks = 8;
constexpr int kTransThreads = 512;
__global__ void __launch_bounds__(kTransThreads)
    k_pack_transpose(const int32_t* __restrict__ s1_idx, const int64_t* __restrict__ s1_off,
                     const int64_t* __restrict__ koff, const int64_t* __restrict__ bt_off, int32_t* __restrict__ bt_ptr,
                     int32_t* __restrict__ bt_perm, int* err) {
  extern __shared__ int32_t s_mem[];
  __shared__ int s_nlong, s_listed;
  const int q = blockIdx.x, tid = threadIdx.x;
  const int rows = (int)(koff[q + 1] - koff[q]), E = (int)(s1_off[q + 1] - s1_off[q]);
  const int32_t* __restrict__ idx = s1_idx + s1_off[q];
  int32_t* __restrict__ perm = bt_perm + s1_off[q];
  int32_t* s_next = s_mem;            // [rows + 1]
  int32_t* s_slot = s_mem + rows + 1; // [E]
  for (int i = tid; i <= rows; i += kTransThreads) s_next[i] = 0;
  if (tid == 0) s_nlong = s_listed = 0;
  __syncthreads();
  bool bad = false;
  for (int e = tid; e < E; e += kTransThreads) {
    const int32_t r = idx[e];
    if (r >= 0 && r < rows) atomicAdd(&s_next[r], 1);
    else bad = true;
  }
  if (bad) atomicOr(err, 16);
  __syncthreads();
  int base = 0;
  for (int i0 = 0; i0 < rows; i0 += kTransThreads) {
    const int i = i0 + tid;
    const int c = i < rows ? s_next[i] : 0;
    int tot;
    const int at = base + block_exscan(c, &tot);
    if (i < rows) {
      s_next[i] = at;
      bt_ptr[bt_off[q] + i] = at;
    }
    base += tot;
  }
  if (tid == 0) bt_ptr[bt_off[q] + rows] = base;
  __syncthreads();
  for (int e = tid; e < E; e += kTransThreads) {
    const int32_t r = idx[e];
    if (r >= 0 && r < rows) s_slot[atomicAdd(&s_next[r], 1)] = e;
  }
  __syncthreads();
  // s_next[r] is now the end of row r
  for (int r = tid; r < rows; r += kTransThreads) {
    const int a = r > 0 ? s_next[r - 1] : 0, b = s_next[r];
    if (b - a > kSortLane) {
      atomicAdd(&s_nlong, 1);
      continue;
    }
    for (int i = a + 1; i < b; ++i) {
      const int32_t v = s_slot[i];
      int k = i;
      for (; k > a && s_slot[k - 1] > v; --k) s_slot[k] = s_slot[k - 1];
      s_slot[k] = v;
    }
  }
  __syncthreads();
  for (int i = tid; i < base; i += kTransThreads) perm[i] = s_slot[i];
  if (s_nlong == 0) return;  // (uniform)
  // the slots are all in perm: their place holds the bitmap, then the list of
  // the long rows (E > kSortLane of them at least)
  __syncthreads();
  const int words = (E + 31) / 32;
  uint32_t* s_bits = reinterpret_cast<uint32_t*>(s_slot);
  int32_t* s_long = s_slot + words;
  for (int r = tid; r < rows; r += kTransThreads)
    if (s_next[r] - (r > 0 ? s_next[r - 1] : 0) > kSortLane) s_long[atomicAdd(&s_listed, 1)] = r;
  for (int g = 0; g < s_nlong; ++g) {
    for (int i = tid; i < words; i += kTransThreads) s_bits[i] = 0;
    __syncthreads();
    const int r = s_long[g], a = r > 0 ? s_next[r - 1] : 0, b = s_next[r];
    for (int i = a + tid; i < b; i += kTransThreads) atomicOr(&s_bits[perm[i] >> 5], 1u << (perm[i] & 31));
    __syncthreads();
    int at = a;
    for (int w0 = 0; w0 < words; w0 += kTransThreads) {
      uint32_t bits = w0 + tid < words ? s_bits[w0 + tid] : 0u;
      int tot;
      int o = at + block_exscan((int)__popc(bits), &tot);
      for (; bits != 0; bits &= bits - 1u) perm[o++] = (w0 + tid) * 32 + __ffs(bits) - 1;
      at += tot;
    }
    __syncthreads();
  }
}

// Per-rank transpose arrays from that grouping (pack rows of rank q occupy
// [koff[q], koff[q+1]) and its slots [s1_off[q], s1_off[q+1])).
__global__ void k_local_bt_ptr(const int32_t* __restrict__ gptr, const int64_t* __restrict__ bt_off,
                               const int64_t* __restrict__ koff, const int64_t* __restrict__ s1_off, int R,
                               int64_t total, int32_t* bt_ptr) {
  for_ranked(total, bt_off, R, [&](int64_t i, int q) {
    const int64_t li = i - bt_off[q];
    bt_ptr[i] = (int32_t)(gptr[koff[q] + li] - s1_off[q]);
  });
}

__global__ void k_local_bt_perm(const int32_t* __restrict__ gperm, int64_t E, const int64_t* __restrict__ s1_off,
                                int R, int32_t* bt_perm) {
  for_ranked(E, s1_off, R, [&](int64_t k, int q) { bt_perm[k] = (int32_t)(gperm[k] - s1_off[q]); });
}

// ---------------------------------------------------------------------------
// Host helpers
// ---------------------------------------------------------------------------
int err_of(int h, const char* what) {
  if (h & 1) return fail(HX_ERR_RANGE, "%s: a column index is outside [0, n)", what);
  if (h & 8) return fail(HX_ERR_ARG, "%s: row_ptr is not non-decreasing", what);
  if (h & 2) return fail(HX_ERR_RANGE, "%s: a rank's halo is not strictly increasing", what);
  if (h & 4) return fail(HX_ERR_RANGE, "%s: a halo column is owned by its own rank", what);
  if (h & 16) return fail(HX_ERR_RANGE, "%s: an index is outside its range", what);
  if (h & 32) return fail(HX_ERR_HIP, "%s: internal error: a list entry fell outside its list", what);
  return HX_SUCCESS;
}

// Copies n values of 64 bits back (ordered after the work on s).
int to_host64(const void* d, int64_t n, std::vector<int64_t>* out, hipStream_t s) {
  out->resize((size_t)n);
  if (n) HX_HIP(hipMemcpyAsync(out->data(), d, (size_t)n * 8, hipMemcpyDeviceToHost, s));
  HX_HIP(hipStreamSynchronize(s));
  return HX_SUCCESS;
}

std::vector<int64_t> prefix(const std::vector<int64_t>& v) {
  std::vector<int64_t> o(v.size() + 1, 0);
  for (size_t i = 0; i < v.size(); ++i) o[i + 1] = o[i] + v[i];
  return o;
}

struct Dense {
  DevMem A, P;
  std::vector<int64_t> sum, nnz;  // host per-row sums and nonzero counts
};

// Prefix sums of a dense R x R table, its row sums (stat[0 .. R)) and nonzero
// counts (stat[R .. 2 R)).
int dense_prefix(Dense* t, int R, int64_t* stat, hipStream_t s) {
  HX_TRY(t->P.alloc((size_t)R * R * 4));
  hipLaunchKernelGGL(k_row_exscan, dim3(R), dim3(TB), 0, s, t->A.as<int32_t>(), t->P.as<int32_t>(), R, stat, stat + R);
  HX_HIP(hipGetLastError());
  return HX_SUCCESS;
}

// Those sums and counts, copied back.
int dense_stats(Dense* t, int R, const int64_t* stat) {
  t->sum.assign(stat, stat + R);
  t->nnz.assign(stat + R, stat + 2 * R);
  for (int64_t v : t->sum)
    if (v >= INT32_MAX) return fail(HX_ERR_UNSUPPORTED, "a rank's list exceeds 2^31 entries");
  return HX_SUCCESS;
}

// Emits the (procs, counts, displs) lists of the rows of a dense table, whose
// offsets are off (off_d on the device).
int dense_lists(const Dense& t, int R, const std::vector<int64_t>& off, const int64_t* off_d, hipStream_t s,
                hx_plan* p, int f_procs) {
  const int64_t tot = off.back();
  for (int k = 0; k < 3; ++k) {
    p->off[f_procs + k] = off;
    HX_TRY(p->d[f_procs + k].alloc((size_t)tot * 4));
  }
  if (tot > 0) {
    hipLaunchKernelGGL(k_row_compact, dim3(R), dim3(TB), 0, s, t.A.as<int32_t>(), t.P.as<int32_t>(), R, off_d,
                       p->d[f_procs].as<int32_t>(), p->d[f_procs + 1].as<int32_t>(), p->d[f_procs + 2].as<int32_t>());
    HX_HIP(hipGetLastError());
  }
  return HX_SUCCESS;
}

int dense_transpose(const DevMem& A, DevMem* AT, int R, hipStream_t s) {
  HX_TRY(AT->alloc((size_t)R * R * 4));
  dim3 g((R + 31) / 32, (R + 31) / 32), b(32, 8);
  hipLaunchKernelGGL(k_transpose, g, b, 0, s, A.as<int32_t>(), AT->as<int32_t>(), R);
  HX_HIP(hipGetLastError());
  return HX_SUCCESS;
}

int zeros(DevMem* d, size_t bytes, hipStream_t s) {
  HX_TRY(d->alloc(bytes));
  if (bytes) HX_HIP(hipMemsetAsync(d->p, 0, bytes, s));
  return HX_SUCCESS;
}

// Builds every plan array from the halos of all ranks (device hcol, host
// offsets; hoff_d: the offsets on the device, uploaded here when empty).
int build_from_halos(hx_plan* p, DevMem& hcol, const std::vector<int64_t>& hoff, DevMem& hoff_d, int check,
                     hipStream_t s) {
  const int R = p->R;
  const int ppn = p->ppn;
  const int64_t n = p->n;
  const int64_t nH = hoff.back();
  const bool loc = p->variant != HX_PLAIN;
  const int v3 = p->variant == HX_LOCALITY_3STEP ? 1 : 0;
  const int NN = (R + ppn - 1) / ppn;
  const Place PL{R, ppn, NN, p->node_map == HX_NODES_CYCLIC ? 1 : 0};
  const int64_t W = (n + 31) / 32;
  const int64_t W1 = W + 1;

  // what the host needs of the tables, read back twice: [error word | sums and
  // nonzero counts of M | of S1 | R1 | S2 | R2]
  DevMem hrank, own, stat;
  HX_TRY(stat.alloc((size_t)(1 + 10 * (int64_t)R) * 8));
  int* err = stat.as<int>();
  int64_t* const st = stat.as<int64_t>() + 1;
  if (!hoff_d.p) HX_TRY(upload_vec(hoff_d, hoff));
  HX_TRY(hrank.alloc((size_t)nH * 4));
  HX_TRY(own.alloc((size_t)nH * 4));
  HX_HIP(hipMemsetAsync(err, 0, 8, s));
  Dense M;
  HX_TRY(zeros(&M.A, (size_t)R * R * 4, s));
  if (nH > 0) {
    hipLaunchKernelGGL(k_entry_info, dim3(walk_blocks(nH)), dim3(TB), 0, s, hcol.as<int32_t>(), nH,
                       hoff_d.as<int64_t>(), p->row_starts_d.as<int64_t>(), R, n, check, hrank.as<int32_t>(),
                       own.as<int32_t>(), M.A.as<int32_t>(), err);
    HX_HIP(hipGetLastError());
  }
  HX_TRY(dense_prefix(&M, R, st, s));
  DevMem MT;
  HX_TRY(dense_transpose(M.A, &MT, R, s));
  std::vector<int64_t> back;
  HX_TRY(to_host64(stat.p, 1 + 2 * (int64_t)R, &back, s));
  HX_TRY(err_of((int)back[0], "halo"));
  HX_TRY(dense_stats(&M, R, back.data() + 1));

  // halo field
  p->off[HX_F_HALO] = hoff;
  p->off[HX_F_UNPACK_SRC] = hoff;
  p->d[HX_F_HALO] = std::move(hcol);

  // node bitmaps (locality)
  DevMem NB, NBP, MD;
  Dense S1, R1, S2, R2;
  DevMem QP;
  if (loc) {
    HX_TRY(NB.alloc((size_t)NN * W1 * 4));
    // the scan runs over the rows of all nodes at once: only differences
    // within a row are used
    DevMem part;
    HX_TRY(NBP.alloc((size_t)(NN * W1 + 1) * 4));
    HX_TRY(part.alloc((size_t)scan_parts(NN * W1) * 8));
    // segments: about 1024 workgroups where the columns allow it
    int seg_bits = kSegBitsMax;
    while (seg_bits > kSegBitsMin && (((W1 * 32) >> seg_bits) + 1) * NN < 1024) --seg_bits;
    const int64_t nseg = (W1 * 32 + ((int64_t)1 << seg_bits) - 1) >> seg_bits;
    hipLaunchKernelGGL(k_node_mark, dim3((unsigned)(nseg * NN)), dim3(512), (size_t)4 << (seg_bits - 5), s,
                       p->d[HX_F_HALO].as<int32_t>(), hoff_d.as<int64_t>(), PL, seg_bits, NB.as<uint32_t>(), W1);
    HX_HIP(hipGetLastError());
    HX_TRY(scan_launch<true>(NB.as<int32_t>(), NBP.as<int32_t>(), NN * W1, part.as<int64_t>(), s));
    HX_TRY(MD.alloc((size_t)NN * R * 4));
    hipLaunchKernelGGL(k_dedup_counts, dim3(blocks_for((int64_t)NN * R)), dim3(TB), 0, s, NB.as<uint32_t>(),
                       NBP.as<int32_t>(), W1, p->row_starts_d.as<int64_t>(), PL, v3, MD.as<int32_t>());
    HX_HIP(hipGetLastError());
    HX_TRY(S1.A.alloc((size_t)R * R * 4));
    hipLaunchKernelGGL(k_stage1_sizes, dim3(blocks_for((int64_t)R * R)), dim3(TB), 0, s, MT.as<int32_t>(),
                       MD.as<int32_t>(), PL, v3, S1.A.as<int32_t>());
    HX_HIP(hipGetLastError());
    HX_TRY(S2.A.alloc((size_t)R * R * 4));
    hipLaunchKernelGGL(k_stage2_sizes, dim3(blocks_for((int64_t)R * R)), dim3(TB), 0, s, M.A.as<int32_t>(), PL,
                       v3, S2.A.as<int32_t>());
    HX_HIP(hipGetLastError());
    HX_TRY(zeros(&QP, (size_t)R * R * 4, s));
    hipLaunchKernelGGL(k_class_prefix, dim3(blocks_for((int64_t)R * ppn)), dim3(TB), 0, s, M.A.as<int32_t>(), PL,
                       v3, QP.as<int32_t>());
    HX_HIP(hipGetLastError());
    HX_TRY(dense_transpose(S1.A, &R1.A, R, s));
    HX_TRY(dense_transpose(S2.A, &R2.A, R, s));
    HX_TRY(dense_prefix(&S1, R, st + 2 * R, s));
    HX_TRY(dense_prefix(&R1, R, st + 4 * R, s));
    HX_TRY(dense_prefix(&S2, R, st + 6 * R, s));
    HX_TRY(dense_prefix(&R2, R, st + 8 * R, s));
    HX_TRY(to_host64(st + 2 * R, 8 * (int64_t)R, &back, s));
    HX_TRY(dense_stats(&S1, R, back.data()));
    HX_TRY(dense_stats(&R1, R, back.data() + 2 * R));
    HX_TRY(dense_stats(&S2, R, back.data() + 4 * R));
    HX_TRY(dense_stats(&R2, R, back.data() + 6 * R));
  } else {
    S1.A = std::move(MT);
    HX_TRY(dense_prefix(&S1, R, st + 2 * R, s));
    HX_TRY(to_host64(st + 2 * R, 2 * (int64_t)R, &back, s));
    HX_TRY(dense_stats(&S1, R, back.data()));
    // stage-1 receive = M (its prefix sums are the receive displacements)
    R1.A = std::move(M.A);
    R1.P = std::move(M.P);
    R1.sum = M.sum;
    R1.nnz = M.nnz;
  }

  // offsets of every list
  std::vector<int64_t> s1_off = prefix(S1.sum);
  std::vector<int64_t> s2_off, r1_tot = R1.sum;
  p->off[HX_F_S1_IDX] = s1_off;
  p->off[HX_F_BT_PERM] = s1_off;
  if (loc) {
    s2_off = prefix(S2.sum);
  } else {
    std::vector<int64_t> z((size_t)R + 1, 0);
    for (int f : {HX_F_S2_PROCS, HX_F_S2_COUNTS, HX_F_S2_DISPLS, HX_F_R2_PROCS, HX_F_R2_COUNTS, HX_F_R2_DISPLS})
      p->off[f] = z;
    s2_off = z;
  }
  p->off[HX_F_S2_SRC] = s2_off;
  p->r1_off = prefix(R1.sum);
  p->r2_off = loc ? prefix(R2.sum) : std::vector<int64_t>((size_t)R + 1, 0);

  const int64_t E1 = s1_off.back(), E2 = s2_off.back();
  if (E1 >= INT32_MAX || E2 >= INT32_MAX || nH >= INT32_MAX)
    return fail(HX_ERR_UNSUPPORTED, "plan lists beyond 2^31 entries");
  // rows of the pack map's transpose: a rank's own rows, its node's for the 3-step plan
  std::vector<int64_t> pack_rows((size_t)R);
  for (int q = 0; q < R; ++q) {
    const int nq = q / ppn;
    pack_rows[q] = v3 ? p->row_starts[std::min(R, (nq + 1) * ppn)] - p->row_starts[nq * ppn]
                      : p->row_starts[q + 1] - p->row_starts[q];
  }
  const std::vector<int64_t> koff = prefix(pack_rows);
  if (koff.back() >= INT32_MAX) return fail(HX_ERR_UNSUPPORTED, "pack-transpose key space beyond 2^31");
  std::vector<int64_t> bt_off((size_t)R + 1, 0);
  for (int q = 0; q < R; ++q) bt_off[q + 1] = bt_off[q] + pack_rows[q] + 1;
  p->off[HX_F_BT_PTR] = bt_off;
  const std::vector<int64_t> l_s1 = prefix(S1.nnz), l_r1 = prefix(R1.nnz), l_s2 = prefix(S2.nnz), l_r2 = prefix(R2.nnz);
  HostPack up;
  const size_t at_s1 = up.add(s1_off), at_s2 = up.add(s2_off), at_r1 = up.add(r1_tot), at_bt = up.add(bt_off),
               at_k = up.add(koff), at_ls1 = up.add(l_s1), at_lr1 = up.add(l_r1), at_ls2 = up.add(l_s2),
               at_lr2 = up.add(l_r2);
  HX_TRY(up.upload());
  const int64_t *s1o_d = up.at<int64_t>(at_s1), *s2o_d = up.at<int64_t>(at_s2), *r1t_d = up.at<int64_t>(at_r1),
                *bto_d = up.at<int64_t>(at_bt), *koff_d = up.at<int64_t>(at_k);
  // lists
  HX_TRY(dense_lists(S1, R, l_s1, up.at<int64_t>(at_ls1), s, p, HX_F_S1_PROCS));
  HX_TRY(dense_lists(R1, R, l_r1, up.at<int64_t>(at_lr1), s, p, HX_F_R1_PROCS));
  if (loc) {
    HX_TRY(dense_lists(S2, R, l_s2, up.at<int64_t>(at_ls2), s, p, HX_F_S2_PROCS));
    HX_TRY(dense_lists(R2, R, l_r2, up.at<int64_t>(at_lr2), s, p, HX_F_R2_PROCS));
  }
  HX_TRY(p->d[HX_F_S1_IDX].alloc((size_t)E1 * 4));
  HX_TRY(p->d[HX_F_S2_SRC].alloc((size_t)E2 * 4));
  HX_TRY(p->d[HX_F_UNPACK_SRC].alloc((size_t)nH * 4));
  const int32_t* PM = loc ? M.P.as<int32_t>() : R1.P.as<int32_t>();
  auto table = [&](const DevMem& d) { return loc ? d.as<int32_t>() : nullptr; };
  if (nH > 0)
    hipLaunchKernelGGL(k_entry_lists, dim3(blocks_for(nH)), dim3(TB), 0, s, p->d[HX_F_HALO].as<int32_t>(),
                       hrank.as<int32_t>(), own.as<int32_t>(), nH, hoff_d.as<int64_t>(),
                       p->row_starts_d.as<int64_t>(), PL, loc ? 1 : 0, v3, S1.P.as<int32_t>(), table(S2.P), table(QP),
                       PM, R1.P.as<int32_t>(), table(R2.P), (const uint32_t*)table(NB), table(NBP), W1, s1o_d, s2o_d,
                       r1t_d, p->d[HX_F_S1_IDX].as<int32_t>(), p->d[HX_F_S2_SRC].as<int32_t>(),
                       p->d[HX_F_UNPACK_SRC].as<int32_t>(), err);
  if (loc && NN * W > 0)
    hipLaunchKernelGGL(k_s1_agg, dim3(blocks_for((int64_t)NN * W)), dim3(TB), 0, s, NB.as<uint32_t>(),
                       NBP.as<int32_t>(), W1, W, p->row_starts_d.as<int64_t>(), PL, v3, S1.P.as<int32_t>(), s1o_d,
                       p->d[HX_F_S1_IDX].as<int32_t>(), err);
  HX_HIP(hipGetLastError());
  // transpose of the pack map, per rank over its pack rows
  HX_TRY(p->d[HX_F_BT_PTR].alloc((size_t)bt_off.back() * 4));
  HX_TRY(p->d[HX_F_BT_PERM].alloc((size_t)E1 * 4));
  // in LDS where every rank's fits (and there are ranks enough to fill the chip)
  int64_t lds = 0;
  for (int q = 0; q < R; ++q) lds = std::max(lds, 4 * (pack_rows[q] + 1 + s1_off[q + 1] - s1_off[q]));
  const bool in_lds = lds <= device_lds_per_block() - 1024 && R >= kTransMinRanks;
  if (in_lds)
    hipLaunchKernelGGL(k_pack_transpose, dim3(R), dim3(kTransThreads), (size_t)lds, s,
                       p->d[HX_F_S1_IDX].as<int32_t>(), s1o_d, koff_d, bto_d, p->d[HX_F_BT_PTR].as<int32_t>(),
                       p->d[HX_F_BT_PERM].as<int32_t>(), err);
  DevMem keys, gptr, gperm;
  if (!in_lds) {
    HX_TRY(keys.alloc((size_t)E1 * 4));
    HX_TRY(gptr.alloc((size_t)(koff.back() + 1) * 4));
    HX_TRY(gperm.alloc((size_t)E1 * 4));
    if (E1 > 0)
      hipLaunchKernelGGL(k_pack_keys, dim3(walk_blocks(E1)), dim3(TB), 0, s, p->d[HX_F_S1_IDX].as<int32_t>(), E1,
                         s1o_d, koff_d, R, keys.as<int32_t>(), err);
  }
  HX_HIP(hipGetLastError());
  HX_TRY(to_host64(stat.p, 1, &back, s));
  HX_TRY(err_of((int)back[0], "plan lists"));
  if (in_lds) return HX_SUCCESS;
  HX_TRY(dev_group_by_key(keys.as<int32_t>(), E1, koff.back(), gptr.as<int32_t>(), gperm.as<int32_t>(), s, true));
  hipLaunchKernelGGL(k_local_bt_ptr, dim3(walk_blocks(bt_off.back())), dim3(TB), 0, s, gptr.as<int32_t>(), bto_d,
                     koff_d, s1o_d, R, bt_off.back(), p->d[HX_F_BT_PTR].as<int32_t>());
  HX_HIP(hipGetLastError());
  if (E1 > 0) {
    hipLaunchKernelGGL(k_local_bt_perm, dim3(walk_blocks(E1)), dim3(TB), 0, s, gperm.as<int32_t>(), E1, s1o_d, R,
                       p->d[HX_F_BT_PERM].as<int32_t>());
    HX_HIP(hipGetLastError());
  }
  HX_HIP(hipStreamSynchronize(s));
  return HX_SUCCESS;
}

int plan_common_checks(int nranks, const int64_t* row_starts, const hx_info* info, hx_plan** out) {
  if (!out) return fail(HX_ERR_ARG, "null out");
  *out = nullptr;
  if (!info) return fail(HX_ERR_ARG, "null info");
  if (nranks <= 0 || !row_starts) return fail(HX_ERR_ARG, "bad nranks / row_starts");
  if (nranks > HX_PLAN_MAX_RANKS) return fail(HX_ERR_UNSUPPORTED, "more than %d ranks", HX_PLAN_MAX_RANKS);
  const int variant = info->variant;
  if (variant != HX_PLAIN && variant != HX_LOCALITY_2STEP && variant != HX_LOCALITY_3STEP)
    return fail(HX_ERR_ARG, "bad variant");
  if (info->ppn < 1) return fail(HX_ERR_ARG, "ppn must be >= 1");
  if (info->node_map != HX_NODES_BLOCK && info->node_map != HX_NODES_CYCLIC)
    return fail(HX_ERR_ARG, "bad node map");
  if (variant == HX_LOCALITY_3STEP && info->node_map != HX_NODES_BLOCK)
    return fail(HX_ERR_UNSUPPORTED, "the 3-step variant needs block placement (a node's rows contiguous)");
  if (row_starts[0] != 0) return fail(HX_ERR_ARG, "row_starts[0] must be 0");
  for (int r = 0; r < nranks; ++r)
    if (row_starts[r + 1] < row_starts[r]) return fail(HX_ERR_ARG, "row_starts must be non-decreasing");
  if (row_starts[nranks] >= INT32_MAX) return fail(HX_ERR_UNSUPPORTED, "more than 2^31 rows");
  return HX_SUCCESS;
}

int plan_alloc(int nranks, const int64_t* row_starts, const hx_info* info, std::unique_ptr<hx_plan>* p) {
  p->reset(new (std::nothrow) hx_plan);
  if (!*p) return fail(HX_ERR_NOMEM, "out of host memory");
  (*p)->R = nranks;
  // more ranks per node than ranks is one node of every rank (under either
  // map); clamping keeps every node-index product inside int
  (*p)->ppn = std::min(info->ppn, nranks);
  (*p)->node_map = info->node_map;
  (*p)->variant = info->variant;
  (*p)->n = row_starts[nranks];
  (*p)->row_starts.assign(row_starts, row_starts + nranks + 1);
  HX_TRY(upload_vec((*p)->row_starts_d, (*p)->row_starts));
  return HX_SUCCESS;
}

}  // namespace

// ---------------------------------------------------------------------------
// Exported device utilities
// ---------------------------------------------------------------------------
int dev_exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, hipStream_t s) {
  DevMem part;
  HX_TRY(part.alloc((size_t)scan_parts(n) * 8));
  HX_TRY(scan_launch(in, out, n, part.as<int64_t>(), s));
  HX_HIP(hipStreamSynchronize(s));
  return HX_SUCCESS;
}

int dev_group_by_key(const int32_t* keys, int64_t n, int64_t nkeys, int32_t* ptr, int32_t* perm, hipStream_t s,
                     bool checked) {
  DevMem work;
  const int32_t* sorted = keys;
  int* err = nullptr;
  if (n > 0) {
    // as few digits as RS_MAX_BITS allows, of even width
    int key_bits = 1;
    while (key_bits < 31 && ((int64_t)1 << key_bits) < nkeys) ++key_bits;
    const int passes = (key_bits + RS_MAX_BITS - 1) / RS_MAX_BITS;
    const int bits = (key_bits + passes - 1) / passes;
    const int nblocks = (int)((n + RS_BLOCK - 1) / RS_BLOCK);
    const int64_t table = ((int64_t)nblocks) << bits;
    // one workspace: [scan partials | error word | keys, twice | values | histogram | its scan]
    const int64_t np = scan_parts(table), nk = passes > 1 ? 2 * n : n, nv = passes > 1 ? n : 0;
    HX_TRY(work.alloc((size_t)(8 * np + 4 * (2 + nk + nv + 2 * table + 1))));
    int64_t* part = work.as<int64_t>();
    err = reinterpret_cast<int*>(part + np);
    int32_t* kbuf = err + 2;
    int32_t* vbuf = kbuf + nk;
    int32_t* hist = vbuf + nv;
    int32_t* offs = hist + table;
    if (!checked) HX_HIP(hipMemsetAsync(err, 0, 4, s));
    const int32_t* vals = nullptr;
    for (int p = 0; p < passes; ++p) {
      // the values end in perm: they alternate between perm and vbuf backwards from the last pass
      int32_t* vout = (passes - 1 - p) % 2 == 0 ? perm : vbuf;
      int32_t* kout = kbuf + (p % 2) * n;
      hipLaunchKernelGGL(k_radix_hist, dim3(nblocks), dim3(TB), 0, s, sorted, n, nkeys, p * bits, bits, hist,
                         nblocks, p == 0 && !checked ? err : nullptr);
      HX_HIP(hipGetLastError());
      HX_TRY(scan_launch(hist, offs, table, part, s));
      hipLaunchKernelGGL(k_radix_scatter, dim3(nblocks), dim3(TB), 0, s, sorted, vals, n, p * bits, bits, offs,
                         nblocks, kout, vout);
      HX_HIP(hipGetLastError());
      sorted = kout;
      vals = vout;
    }
  }
  hipLaunchKernelGGL(k_group_ptr, dim3(blocks_for(std::max(n, (nkeys + 1) / 4), CHUNK)), dim3(TB), 0, s, sorted, n,
                     nkeys, ptr, checked ? nullptr : err);
  HX_HIP(hipGetLastError());
  if (err && !checked) {
    int h = 0;
    HX_HIP(hipMemcpyAsync(&h, err, sizeof h, hipMemcpyDeviceToHost, s));
    HX_HIP(hipStreamSynchronize(s));
    return err_of(h, "grouping");
  }
  HX_HIP(hipStreamSynchronize(s));
  return HX_SUCCESS;
}

int dev_check_range(const int32_t* idx, int64_t n, int64_t hi, const char* what, hipStream_t s) {
  if (n <= 0) return HX_SUCCESS;
  DevMem err;
  HX_TRY(zeros(&err, 8, s));
  hipLaunchKernelGGL(k_check_range, dim3(blocks_for(n)), dim3(TB), 0, s, idx, n, hi, err.as<int>());
  HX_HIP(hipGetLastError());
  std::vector<int64_t> back;
  HX_TRY(to_host64(err.p, 1, &back, s));
  return err_of((int)back[0], what);
}

int dev_count_nonempty(const int32_t* ptr, int64_t n, unsigned long long* acc, hipStream_t s) {
  if (n <= 0) return HX_SUCCESS;
  hipLaunchKernelGGL(k_count_nonempty, dim3(std::min(blocks_for(n), 512u)), dim3(TB), 0, s, ptr, n, acc);
  HX_HIP(hipGetLastError());
  return HX_SUCCESS;
}

int dev_count_distinct(const int32_t* idx, int64_t n, int64_t domain, DevMem* flags, unsigned long long* acc,
                       hipStream_t s) {
  if (n <= 0 || domain <= 0) return HX_SUCCESS;
  const int64_t nwords = (domain + 3) / 4;
  HX_TRY(zeros(flags, (size_t)nwords * 4, s));
  hipLaunchKernelGGL(k_flag, dim3(blocks_for(n)), dim3(TB), 0, s, idx, n, domain, flags->as<unsigned char>());
  HX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_count_flags, dim3(std::min(blocks_for(nwords), 512u)), dim3(TB), 0, s, flags->as<uint32_t>(),
                     nwords, acc);
  HX_HIP(hipGetLastError());
  return HX_SUCCESS;
}

}  // namespace hx

using namespace hx;

// ===========================================================================
// Public plan API
// ===========================================================================
extern "C" int hx_plan_from_csr(int nranks, const int64_t* row_starts, const hx_info* info,
                                const int64_t* row_ptr, const int32_t* cols, void* stream, hx_plan** out) {
  HX_TRY(plan_common_checks(nranks, row_starts, info, out));
  const int64_t n = row_starts[nranks];
  if (n > 0 && !row_ptr) return fail(HX_ERR_ARG, "null row_ptr");
  hipStream_t s = (hipStream_t)stream;
  std::unique_ptr<hx_plan> p;
  HX_TRY(plan_alloc(nranks, row_starts, info, &p));
  const int64_t W = (n + 127) / 128 * 4;  // words of a bitmap row (whole 16-byte vectors)
  // Halo discovery marks one bit per (rank, column).  The bitmaps of a group
  // of ranks are built, counted and compacted before the next group, so the
  // bitmap memory stays within a budget whatever the rank count.
  int64_t budget = (int64_t)1 << 30;
  if (const char* e = std::getenv("HX_PLAN_BITMAP_BYTES")) budget = std::max<int64_t>(1, std::atoll(e));
  const int64_t group = std::max<int64_t>(1, std::min<int64_t>(nranks, budget / std::max<int64_t>(W * 4, 1)));
  DevMem B, cnt, ent;  // cnt: [error word | set bits of each rank of the group]
  HX_TRY(B.alloc((size_t)std::max<int64_t>(group * W * 4, 4)));
  HX_TRY(cnt.alloc((size_t)(group + 1) * 8));
  int* err = cnt.as<int>();
  unsigned long long* bits = cnt.as<unsigned long long>() + 1;
  HX_TRY(ent.alloc((size_t)(group + 1) * 8));
  std::vector<int64_t> hoff(1, 0);
  std::vector<DevMem> parts;
  DevMem off_d;  // the offsets of a group
  for (int r0 = 0; r0 < nranks; r0 += (int)group) {
    const int g = (int)std::min<int64_t>(group, nranks - r0);
    const int64_t i0 = row_starts[r0], rows = row_starts[r0 + g] - i0;
    // a rank's bitmap is built in LDS where a few segments hold it (the
    // entries are streamed once a segment) and there are enough ranks
    const int nseg = (int)std::min<int64_t>((n + ((int64_t)1 << kMarkSegBits) - 1) >> kMarkSegBits, kMarkMaxSegs + 1);
    const int64_t lds = std::min<int64_t>(W * 4, (int64_t)1 << (kMarkSegBits - 3));
    const bool in_lds = rows > 0 && nseg <= kMarkMaxSegs && g >= kMarkMinRanks && lds <= device_lds_per_block() - 1024;
    if (W > 0 && !in_lds) HX_HIP(hipMemsetAsync(B.p, 0, (size_t)g * W * 4, s));
    HX_HIP(hipMemsetAsync(cnt.p, 0, (size_t)(g + 1) * 8, s));
    if (rows > 0) {
      hipLaunchKernelGGL(k_rank_entries, dim3(std::min(blocks_for(std::max<int64_t>(rows, g + 1)), 2048u)), dim3(TB), 0,
                         s, p->row_starts_d.as<int64_t>(), i0, rows, r0, g, row_ptr, ent.as<int64_t>(), err);
      if (in_lds)
        hipLaunchKernelGGL(k_mark_lds, dim3((unsigned)((g + 7) / 8 * 8 * nseg)), dim3(kMarkThreads), (size_t)lds, s,
                           p->row_starts_d.as<int64_t>(), n, r0, g, nseg, ent.as<int64_t>(), cols, B.as<uint32_t>(), W,
                           bits, err);
      else
        hipLaunchKernelGGL(k_mark_csr, dim3((unsigned)(8 * device_cus())), dim3(TB), 0, s,
                           p->row_starts_d.as<int64_t>(), n, r0, g, ent.as<int64_t>(), cols, B.as<uint32_t>(), W,
                           err);
      HX_HIP(hipGetLastError());
    }
    if (!in_lds) {
      hipLaunchKernelGGL(k_popc_rows, dim3(g), dim3(kBitThreads), 0, s, B.as<uint32_t>(), W, (int64_t*)bits);
      HX_HIP(hipGetLastError());
    }
    std::vector<int64_t> hc;
    HX_TRY(to_host64(cnt.p, g + 1, &hc, s));
    HX_TRY(err_of((int)hc[0], "csr"));
    hc.erase(hc.begin());
    std::vector<int64_t> off = prefix(hc);
    if (hoff.back() + off.back() >= INT32_MAX) return fail(HX_ERR_UNSUPPORTED, "total halo beyond 2^31 entries");
    for (int k = 0; k < g; ++k) hoff.push_back(hoff.back() + hc[k]);
    parts.emplace_back();
    if (off.back() > 0) {
      off_d.release();
      HX_TRY(upload_vec(off_d, off));
      HX_TRY(parts.back().alloc((size_t)off.back() * 4));
      hipLaunchKernelGGL(k_compact_bits, dim3(g), dim3(kBitThreads), 0, s, B.as<uint32_t>(), W, off_d.as<int64_t>(),
                         parts.back().as<int32_t>());
      HX_HIP(hipGetLastError());
    }
  }
  B.release();
  DevMem hcol;
  if (parts.size() == 1) {
    hcol = std::move(parts[0]);  // (one group: its offsets are all ranks')
  } else {
    HX_TRY(hcol.alloc((size_t)hoff.back() * 4));
    int64_t at = 0;
    for (DevMem& d : parts) {
      const int64_t len = (int64_t)(d.bytes / 4);
      if (len > 0)
        HX_HIP(hipMemcpyAsync(hcol.as<int32_t>() + at, d.p, (size_t)len * 4, hipMemcpyDeviceToDevice, s));
      at += len;
    }
    HX_HIP(hipStreamSynchronize(s));
    parts.clear();
    off_d.release();
  }
  HX_TRY(build_from_halos(p.get(), hcol, hoff, off_d, 0, s));
  *out = p.release();
  return HX_SUCCESS;
}

extern "C" int hx_plan_from_halos(int nranks, const int64_t* row_starts, const hx_info* info,
                                  const int64_t* halo_ptr, const int32_t* halo_cols, void* stream,
                                  hx_plan** out) {
  HX_TRY(plan_common_checks(nranks, row_starts, info, out));
  if (!halo_ptr) return fail(HX_ERR_ARG, "null halo_ptr");
  if (halo_ptr[0] != 0) return fail(HX_ERR_ARG, "halo_ptr[0] must be 0");
  for (int r = 0; r < nranks; ++r)
    if (halo_ptr[r + 1] < halo_ptr[r]) return fail(HX_ERR_ARG, "halo_ptr must be non-decreasing");
  const int64_t nH = halo_ptr[nranks];
  if (nH >= INT32_MAX) return fail(HX_ERR_UNSUPPORTED, "total halo beyond 2^31 entries");
  if (nH > 0 && !halo_cols) return fail(HX_ERR_ARG, "null halo_cols");
  hipStream_t s = (hipStream_t)stream;
  std::unique_ptr<hx_plan> p;
  HX_TRY(plan_alloc(nranks, row_starts, info, &p));
  DevMem hcol;
  HX_TRY(hcol.alloc((size_t)nH * 4));
  if (nH) HX_HIP(hipMemcpyAsync(hcol.p, halo_cols, (size_t)nH * 4, hipMemcpyDeviceToDevice, s));
  std::vector<int64_t> hoff(halo_ptr, halo_ptr + nranks + 1);
  DevMem hoff_d;
  HX_TRY(build_from_halos(p.get(), hcol, hoff, hoff_d, 1, s));
  *out = p.release();
  return HX_SUCCESS;
}

extern "C" int hx_plan_free(hx_plan** p) {
  if (!p) return HX_SUCCESS;
  delete *p;
  *p = nullptr;
  return HX_SUCCESS;
}

extern "C" int hx_plan_field_size(const hx_plan* p, int rank, hx_field f, int64_t* count) {
  if (!p || !count) return fail(HX_ERR_ARG, "null argument");
  if (rank < 0 || rank >= p->R || (int)f < 0 || f >= HX_F_COUNT) return fail(HX_ERR_RANGE, "bad rank or field");
  *count = p->size(f, rank);
  return HX_SUCCESS;
}

extern "C" int hx_plan_describe(const hx_plan* p, int* nranks, int64_t* n, hx_info* info, int64_t* row_starts) {
  if (!p) return fail(HX_ERR_ARG, "null plan");
  if (nranks) *nranks = p->R;
  if (n) *n = p->n;
  if (info) {
    info->variant = p->variant;
    info->ppn = p->ppn;
    info->node_map = p->node_map;
  }
  if (row_starts) std::copy(p->row_starts.begin(), p->row_starts.end(), row_starts);
  return HX_SUCCESS;
}

extern "C" int hx_plan_field_all(const hx_plan* p, hx_field f, int64_t* offsets, int32_t* dst) {
  if (!p) return fail(HX_ERR_ARG, "null plan");
  if ((int)f < 0 || f >= HX_F_COUNT) return fail(HX_ERR_RANGE, "bad field");
  if (offsets) std::copy(p->off[f].begin(), p->off[f].end(), offsets);
  const int64_t c = p->tot(f);
  if (dst && c > 0) HX_HIP(hipMemcpy(dst, p->d[f].p, (size_t)c * 4, hipMemcpyDeviceToHost));
  return HX_SUCCESS;
}

extern "C" int hx_plan_field_copy(const hx_plan* p, int rank, hx_field f, int32_t* dst) {
  int64_t c = 0;
  HX_TRY(hx_plan_field_size(p, rank, f, &c));
  if (c == 0) return HX_SUCCESS;
  if (!dst) return fail(HX_ERR_ARG, "null destination");
  HX_HIP(hipMemcpy(dst, p->d[f].as<int32_t>() + p->off[f][rank], (size_t)c * 4, hipMemcpyDeviceToHost));
  return HX_SUCCESS;
}

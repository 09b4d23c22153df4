// Launch tables of the data-movement kernels: the job table and tile prefix
// in device memory, the launch shape, and the dispatch to the kernel
// translation units (move_gather / move_scatter / move_segsum).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <memory>
#include <new>

#include "common.h"
#include "move_kernels.h"

namespace hx {
namespace {

// outside[j] = how many of job j's indices lie outside its source window
// (rows outside a window are read from global memory, so a window that
// holds few of them only costs its staging).
__global__ void __launch_bounds__(256) k_check_windows(const GatherJob* __restrict__ jobs, int njobs,
                                                       int64_t* __restrict__ outside) {
  __shared__ unsigned long long s_out;
  for (int j = blockIdx.x; j < njobs; j += gridDim.x) {
    const GatherJob g = jobs[j];
    if (threadIdx.x == 0) s_out = 0;
    __syncthreads();
    unsigned long long out = 0;
    if (g.win_rows > 0 && g.idx != nullptr) {
      for (int64_t e = threadIdx.x; e < g.nrows; e += blockDim.x) {
        const int64_t v = g.idx[e];
        out += (v < g.win_lo || v >= g.win_lo + g.win_rows) ? 1 : 0;
      }
    }
    if (out) atomicAdd(&s_out, out);  // LDS atomic
    __syncthreads();
    if (threadIdx.x == 0) outside[j] = (int64_t)s_out;
    __syncthreads();  // s_out is reset for the next job
  }
}

// te[t] = {ptr[r0], ptr[r1]} of tile t of a segmented-sum or push table
// (its rows [r0, r1) of job j), so a workgroup can load its tile's row
// pointers and entry indices together instead of one after the other.
__global__ void __launch_bounds__(256) k_tile_terms(const SegSumJob* __restrict__ jobs,
                                                    const int64_t* __restrict__ ts, int njobs, int64_t ntiles,
                                                    int tile_rows, int2* __restrict__ te) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < ntiles;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int j = kern::job_of(ts, njobs, t);
    const int64_t r0 = (t - ts[j]) * (int64_t)tile_rows;
    const int64_t r1 = min(r0 + (int64_t)tile_rows, jobs[j].nrows);
    te[t] = make_int2(jobs[j].ptr[r0], jobs[j].ptr[r1]);
  }
}

// Total terms of a segmented sum's jobs: the sum of ptr[nrows] - ptr[0].
__global__ void __launch_bounds__(256) k_term_count(const SegSumJob* __restrict__ jobs, int njobs,
                                                    unsigned long long* __restrict__ total) {
  unsigned long long acc = 0;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < njobs; j += gridDim.x * blockDim.x)
    acc += (unsigned long long)(jobs[j].ptr[jobs[j].nrows] - jobs[j].ptr[0]);
  if (acc) atomicAdd(total, acc);
}

// Clears the windows of jobs that hold less than half of their indices
// and marks the jobs whose window holds all of them (device-side count).
int drop_bad_windows(std::vector<GatherJob>* w) {
  std::vector<int> at;
  for (size_t i = 0; i < w->size(); ++i) {
    (*w)[i].win_all = 0;
    if ((*w)[i].win_rows > 0 && (*w)[i].nrows > 0) at.push_back((int)i);
  }
  if (at.empty()) return HX_SUCCESS;
  std::vector<GatherJob> sub;
  for (int i : at) sub.push_back((*w)[i]);
  DevMem d_jobs, d_out;
  HX_TRY(upload_vec(d_jobs, sub));
  HX_TRY(d_out.alloc(sub.size() * sizeof(int64_t)));
  const int grid = (int)std::min<size_t>(sub.size(), 4096);
  hipLaunchKernelGGL(k_check_windows, dim3(grid), dim3(256), 0, 0, d_jobs.as<GatherJob>(), (int)sub.size(),
                     d_out.as<int64_t>());
  HX_HIP(hipGetLastError());
  std::vector<int64_t> outside(sub.size(), 0);
  HX_HIP(hipMemcpy(outside.data(), d_out.p, outside.size() * sizeof(int64_t), hipMemcpyDeviceToHost));
  for (size_t k = 0; k < at.size(); ++k) {
    GatherJob& g = (*w)[at[k]];
    if (g.idx == nullptr || 2 * outside[k] > g.nrows) {
      g.win_lo = 0;
      g.win_rows = 0;
    } else {
      g.win_all = outside[k] == 0 ? 1 : 0;
    }
  }
  return HX_SUCCESS;
}

// Vector width usable for a table: divides row_bytes and every base pointer.
int pick_vec(int row_bytes, uintptr_t align_or) {
  for (int vb : {16, 8, 4}) {
    if (row_bytes % vb == 0 && (align_or % vb) == 0) return vb;
  }
  return 0;
}

// Launch shape of a table (schedule checks, the jobs with rows and their tile
// prefix, vector width, grid); allocates nothing.
template <class J>
int shape_table(const std::vector<J>& jobs, int kind, int dtype, int row_bytes, const Sched& s0, LaunchTable* t,
                uintptr_t align_or, std::vector<J>* kept_out, std::vector<int64_t>* ts_out) {
  t->kind = kind;
  t->dtype = dtype;
  t->row_bytes = row_bytes;
  t->sched = s0;
  t->vec16 = 0;
  if (t->sched.tile_rows <= 0 || t->sched.block_threads <= 0 || t->sched.blocks_per_cu <= 0)
    return fail(HX_ERR_ARG, "invalid schedule (tile_rows %d, block_threads %d, blocks_per_cu %d)",
                t->sched.tile_rows, t->sched.block_threads, t->sched.blocks_per_cu);
  if (t->sched.block_threads != 256 && t->sched.block_threads != 512 &&
      !(kind != KIND_SCATTER && t->sched.block_threads == 1024))
    return fail(HX_ERR_ARG, "block_threads must be 256, 512 or 1024");
  // keep only jobs with rows; tile prefix
  std::vector<J>& kept = *kept_out;
  std::vector<int64_t>& ts = *ts_out;
  kept.clear();
  ts.assign(1, 0);
  for (const J& j : jobs) {
    if (j.nrows <= 0) continue;
    kept.push_back(j);
    ts.push_back(ts.back() + (j.nrows + t->sched.tile_rows - 1) / t->sched.tile_rows);
  }
  t->njobs = (int)kept.size();
  t->ntiles = ts.back();
  if (t->ntiles == 0) {
    t->grid = 0;
    t->jobs.release();
    t->tile_start.release();
    t->tile_terms.release();
    return HX_SUCCESS;
  }
  t->vec_bytes = pick_vec(row_bytes, align_or);
  if (t->vec_bytes == 0) return fail(HX_ERR_ARG, "rows of %d bytes / buffers not 4-byte aligned", row_bytes);
  if (kind == KIND_SEGSUM && (size_t)t->vec_bytes < dtype_bytes(dtype))
    return fail(HX_ERR_ARG, "FP64 buffers must be 8-byte aligned");
  int64_t want = (int64_t)t->sched.blocks_per_cu * device_cus();
  want = std::min<int64_t>(want, (t->ntiles + 7) / 8 * 8);
  want = std::min<int64_t>(want, int64_t(1) << 30);  // a launchable grid; larger tables take tile ranges
  want = std::max<int64_t>(8, (want + 7) / 8 * 8);
  t->grid = (int)want;
  return HX_SUCCESS;
}

// Jobs and tile prefix to the device, in one copy.
template <class J>
int upload_table(const std::vector<J>& kept, const std::vector<int64_t>& ts, LaunchTable* t) {
  if (t->ntiles == 0) return HX_SUCCESS;
  HostPack up;
  up.add(kept);
  // the tile prefix, then every tile's job
  std::vector<int64_t> tiles(ts);
  tiles.resize(ts.size() + ((size_t)t->ntiles + 1) / 2);
  int32_t* job = reinterpret_cast<int32_t*>(tiles.data() + ts.size());
  for (size_t j = 0; j + 1 < ts.size(); ++j) std::fill(job + ts[j], job + ts[j + 1], (int32_t)j);
  const size_t at_ts = up.add(tiles);
  HX_TRY(up.upload());
  t->jobs = std::move(up.dev);
  t->tile_start.borrow(t->jobs.as<char>() + at_ts, tiles.size() * sizeof(int64_t));
  return HX_SUCCESS;
}

template <class J>
int build_table(const std::vector<J>& jobs, int kind, int dtype, int row_bytes, const Sched& s0, LaunchTable* t,
                uintptr_t align_or) {
  std::vector<J> kept;
  std::vector<int64_t> ts;
  HX_TRY(shape_table(jobs, kind, dtype, row_bytes, s0, t, align_or, &kept, &ts));
  return upload_table(kept, ts, t);
}

// Entry range of every tile of a CSR-driven table (segmented sum, push
// pack), read by their staged forms.
int fill_tile_terms(LaunchTable* t) {
  if (t->ntiles == 0) return HX_SUCCESS;
  HX_TRY(t->tile_terms.alloc((size_t)t->ntiles * sizeof(int2)));
  const int grid = (int)std::min<int64_t>((t->ntiles + 255) / 256, 4096);
  hipLaunchKernelGGL(k_tile_terms, dim3(grid), dim3(256), 0, 0, t->jobs.as<SegSumJob>(), t->tile_start.as<int64_t>(),
                     t->njobs, t->ntiles, t->sched.tile_rows, t->tile_terms.as<int2>());
  HX_HIP(hipGetLastError());
  HX_HIP(hipStreamSynchronize(0));
  return HX_SUCCESS;
}

uintptr_t align_of(const std::vector<SegSumJob>& jobs, int row_bytes) {
  uintptr_t a = (uintptr_t)row_bytes;
  for (const auto& j : jobs) {
    if (j.nrows <= 0) continue;
    a |= (uintptr_t)j.in | (uintptr_t)j.out | (uintptr_t)j.out2;
    if (j.in2) a |= (uintptr_t)j.in2;
  }
  return a;
}

}  // namespace

int build_gather_table(const std::vector<GatherJob>& jobs, int dtype, int row_bytes, const Sched& s, LaunchTable* t,
                       int tag) {
  t->tag = tag;
  t->copies.reset();
  bool kinds[2] = {false, false};
  for (const auto& j : jobs)
    if (j.nrows > 0) kinds[j.idx ? 1 : 0] = true;
  if (kinds[0] && kinds[1]) {
    std::vector<GatherJob> indexed, copied;
    for (const auto& j : jobs) (j.idx ? indexed : copied).push_back(j);
    std::unique_ptr<LaunchTable> c(new (std::nothrow) LaunchTable);
    if (!c) return fail(HX_ERR_NOMEM, "out of host memory");
    HX_TRY(build_gather_table(copied, dtype, row_bytes, s, c.get(), tag));
    HX_TRY(build_gather_table(indexed, dtype, row_bytes, s, t, tag));
    t->copies = std::move(c);
    return HX_SUCCESS;
  }
  uintptr_t a = (uintptr_t)row_bytes;
  for (const auto& j : jobs) {
    if (j.nrows <= 0) continue;
    a |= (uintptr_t)j.src | (uintptr_t)j.dst | (uintptr_t)j.dst2;
  }
  // short rows in 16-byte groups per lane: rows of 4 or 8 bytes whose
  // buffers are aligned to the row size, and every index list congruent
  // with its destination (the first row whose destination is 16-byte
  // aligned also aligns the V-wide index loads, V = 16 / row_bytes)
  bool vec = s.pair_rows && (row_bytes == 8 || row_bytes == 4) && (a % (uintptr_t)row_bytes) == 0;
  if (vec) {
    const uintptr_t V = 16 / (uintptr_t)row_bytes;
    for (const auto& j : jobs) {
      if (j.nrows <= 0 || j.idx == nullptr) continue;
      for (const int32_t* ix : {j.idx, j.idx2})
        if (ix && (((uintptr_t)ix % 4) != 0 || ((uintptr_t)ix / 4) % V != ((uintptr_t)j.dst / row_bytes) % V))
          vec = false;
    }
  }
  // source windows: kept where the schedule asks for them and they fit (the
  // 16-byte group form stages from the window's 16-byte aligned start)
  std::vector<GatherJob> w(jobs);
  const int64_t win_cap = std::min<int64_t>(kWinBytes, device_lds_per_block());
  auto win_span = [&](const GatherJob& j) -> int64_t {
    const int64_t bytes = j.win_rows * (int64_t)row_bytes;
    return vec ? bytes + (int64_t)(((uintptr_t)j.src + (uintptr_t)(j.win_lo * row_bytes)) & 15) : bytes;
  };
  for (auto& j : w) {
    if (!s.lds_window || j.idx == nullptr || j.win_rows <= 0 || win_span(j) > win_cap || j.win_lo < 0) {
      j.win_lo = 0;
      j.win_rows = 0;
    }
  }
  HX_TRY(drop_bad_windows(&w));
  int64_t win_bytes = 0;
  for (const auto& j : w) {
    if (j.win_rows <= 0) continue;
    if (!vec) a |= (uintptr_t)(j.src + j.win_lo * (int64_t)row_bytes);
    win_bytes = std::max(win_bytes, win_span(j));
  }
  HX_TRY(build_table(w, KIND_GATHER, dtype, row_bytes, s, t, a));
  // (the runtime-row-size kernel form ignores windows and reads global memory)
  t->win_bytes = t->ntiles > 0 ? (int)((win_bytes + 15) / 16 * 16) : 0;
  t->vec16 = t->ntiles > 0 && vec ? 1 : 0;
  t->partial_win = 0;
  t->identity = 0;
  for (const auto& j : w)
    if (j.nrows > 0 && j.idx == nullptr) t->identity = 1;
  if (t->identity) t->vec16 = 0;
  t->deliver = 1;
  for (const auto& j : w)
    if (j.nrows > 0 && j.dst2 == nullptr) t->deliver = 0;
  if (t->identity && row_bytes / t->vec_bytes > kern::kFlatMaxVec) t->deliver = 0;
  for (const auto& j : w)
    if (j.nrows > 0 && j.win_rows > 0 && !j.win_all) t->partial_win = 1;
  return HX_SUCCESS;
}

// Shape of a segmented-sum table: term windows, launch shape, term buffer
// (no device memory).
// Shape of a segmented sum of rows of one value, one row per lane: each
// job keeps its term window where it fits (80 KiB with the staging's
// alignment) and lies in one input; no term buffer.
int shape_segsum_vec_table(const std::vector<SegSumJob>& jobs, int dtype, int row_bytes, const Sched& s,
                           LaunchTable* t, int tag, std::vector<SegSumJob>* kept, std::vector<int64_t>* ts) {
  t->tag = tag;
  std::vector<SegSumJob> w(jobs);
  const int64_t cap = std::min<int64_t>(kWinBytes, device_lds_per_block());
  int64_t win_bytes = 0;
  for (auto& j : w) {
    const int64_t hi = j.win_lo + j.win_rows;
    const bool one_input = hi <= j.split || j.win_lo >= j.split;
    int64_t span = 0;
    if (j.win_rows > 0 && j.win_lo >= 0 && one_input) {
      const char* a = j.win_lo < j.split ? j.in + j.win_lo * (int64_t)row_bytes
                                         : j.in2 + (j.win_lo - j.split) * (int64_t)row_bytes;
      span = j.win_rows * (int64_t)row_bytes + (int64_t)((uintptr_t)a & 15);
    }
    if (!s.lds_window || j.nrows <= 0 || span <= 0 || span > cap) {
      j.win_lo = j.win_rows = 0;
    } else {
      win_bytes = std::max(win_bytes, span);
    }
  }
  HX_TRY(shape_table(w, KIND_SEGSUM, dtype, row_bytes, s, t, align_of(w, row_bytes), kept, ts));
  t->win_bytes = t->ntiles > 0 ? (int)((win_bytes + 15) / 16 * 16) : 0;
  t->val_bytes = 0;
  t->vec16 = t->ntiles > 0 ? 1 : 0;
  t->vec_depth = 4;  // (set from the jobs' term counts when the table is uploaded)
  return HX_SUCCESS;
}

int shape_segsum_table(const std::vector<SegSumJob>& jobs, int dtype, int row_bytes, const Sched& s,
                       LaunchTable* t, int tag, std::vector<SegSumJob>* kept, std::vector<int64_t>* ts) {
  if (s.pair_rows && (row_bytes == 4 || row_bytes == 8) && (size_t)row_bytes == dtype_bytes(dtype))
    return shape_segsum_vec_table(jobs, dtype, row_bytes, s, t, tag, kept, ts);
  t->tag = tag;
  // term windows: kept where the schedule asks for them, they fit, and they
  // lie inside one of the two inputs
  // (all jobs or none: a job without a window would run the windowed form's
  // row-parallel loop from global memory, slower than the plain form)
  std::vector<SegSumJob> w(jobs);
  const int64_t cap = std::min<int64_t>(kSegWinBytes, device_lds_per_block() - (8 << 10));
  int64_t win_bytes = 0;
  // (the windowed kernel is bounded to 512 lanes)
  bool all = s.lds_window != 0 && s.block_threads <= 512;
  for (const auto& j : w) {
    if (j.nrows <= 0) continue;
    const int64_t bytes = j.win_rows * (int64_t)row_bytes;
    const int64_t hi = j.win_lo + j.win_rows;
    const bool one_input = hi <= j.split || j.win_lo >= j.split;
    if (j.win_rows <= 0 || j.win_lo < 0 || bytes > cap || !one_input) all = false;
    else win_bytes = std::max(win_bytes, bytes);
  }
  if (!all) {
    win_bytes = 0;
    for (auto& j : w) j.win_lo = j.win_rows = 0;
  }
  uintptr_t a = align_of(w, row_bytes);
  for (const auto& j : w)
    if (j.win_rows > 0 && j.nrows > 0)
      a |= (uintptr_t)(j.win_lo < j.split ? j.in + j.win_lo * (int64_t)row_bytes
                                           : j.in2 + (j.win_lo - j.split) * (int64_t)row_bytes);
  HX_TRY(shape_table(w, KIND_SEGSUM, dtype, row_bytes, s, t, a, kept, ts));
  t->win_bytes = t->ntiles > 0 ? (int)win_bytes : 0;
  // term buffer: about two terms per tile row, at least 4 KiB and at most
  // kSegValueBytes, whole rows (small tiles leave LDS for more workgroups);
  // none for tiles that stage no pointers, whose rows add straight from memory
  int64_t vb = std::min<int64_t>(kSegValueBytes, std::max<int64_t>(4096, 2 * (int64_t)s.tile_rows * row_bytes));
  t->val_bytes = t->ntiles > 0 && s.tile_rows <= kStageRows ? (int)(vb / row_bytes * row_bytes) : 0;
  return HX_SUCCESS;
}

// One-value sums: 16 terms per row loaded together (one row per lane) where
// rows average more than three terms (the owner sums of high fan-out packs),
// else 4; further terms are a serial chain (one rank's 1024 rows of 8 terms
// each: 7.7 us with 4, 5.0 with 16).
static int depth_of(int64_t terms, int64_t rows) { return terms > 3 * rows ? 16 : 4; }

int build_segsum_table(const std::vector<SegSumJob>& jobs, int dtype, int row_bytes, const Sched& s,
                       LaunchTable* t, int tag) {
  std::vector<SegSumJob> kept;
  std::vector<int64_t> ts;
  HX_TRY(shape_segsum_table(jobs, dtype, row_bytes, s, t, tag, &kept, &ts));
  if (t->ntiles == 0) return HX_SUCCESS;
  HX_TRY(upload_table(kept, ts, t));
  t->deliver = tag == TAG_FWD_SUM ? 1 : 0;
  for (const auto& j : kept)
    if (j.out2 == nullptr) t->deliver = 0;
  if (t->vec16) {
    int64_t rows = 0;
    for (const auto& j : kept) rows += j.nrows;
    DevMem d_terms;
    HX_TRY(d_terms.alloc(sizeof(unsigned long long)));
    HX_HIP(hipMemset(d_terms.p, 0, sizeof(unsigned long long)));
    const int grid = (int)std::min<size_t>((kept.size() + 255) / 256, 1024);
    hipLaunchKernelGGL(k_term_count, dim3(grid), dim3(256), 0, 0, t->jobs.as<SegSumJob>(), t->njobs,
                       d_terms.as<unsigned long long>());
    HX_HIP(hipGetLastError());
    unsigned long long terms = 0;
    HX_HIP(hipMemcpy(&terms, d_terms.p, sizeof(terms), hipMemcpyDeviceToHost));
    t->vec_depth = depth_of((int64_t)terms, rows);
  }
  return fill_tile_terms(t);
}

int launch_segsum_one(const SegSumJob& job, int64_t terms, int dtype, int row_bytes, const Sched& s,
                      hipStream_t stream) {
  LaunchTable t;
  std::vector<SegSumJob> kept;
  std::vector<int64_t> ts;
  Sched sc = s;
  if (!sc.pair_rows && sc.lds_window) {  // (the windowed form reads launch tables only)
    sc.lds_window = 0;
    sc.tile_rows = std::min(sc.tile_rows, kStageRows);
  }
  HX_TRY(shape_segsum_table(std::vector<SegSumJob>(1, job), dtype, row_bytes, sc, &t, TAG_OWNER_SUM, &kept, &ts));
  if (t.ntiles == 0) return HX_SUCCESS;
  t.vec_depth = depth_of(terms, job.nrows);
  LaunchOpt o;
  o.one = &kept[0];
  return launch_table(t, stream, o);
}

int build_scatter_table(const std::vector<SegSumJob>& jobs, int dtype, int row_bytes, const Sched& s,
                        LaunchTable* t, int tag) {
  t->tag = tag;
  Sched sc = s;
  sc.block_threads = std::min(sc.block_threads, 512);  // the push pack runs at most 512 lanes
  HX_TRY(build_table(jobs, KIND_SCATTER, dtype, row_bytes, sc, t, align_of(jobs, row_bytes)));
  t->deliver = 1;
  for (const auto& j : jobs)
    if (j.nrows > 0 && j.out2 == nullptr) t->deliver = 0;
  return fill_tile_terms(t);
}

int launch_table(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  if (t.ntiles == 0) return HX_SUCCESS;
  if (o.deliver && !t.deliver) return fail(HX_ERR_STATE, "a launch table without second destinations");
  if (t.kind == KIND_GATHER) launch_gather_kernels(t, s, o);
  else if (t.kind == KIND_SCATTER) launch_scatter_kernels(t, s, o);
  else if (o.one) launch_segsum_one_kernels(t, s, o);
  else launch_segsum_kernels(t, s, o);
  HX_HIP(hipGetLastError());
  return t.copies ? launch_table(*t.copies, s, o) : HX_SUCCESS;
}

void split_gather_by_counts(const GatherJob& j, const std::vector<int32_t>& counts, size_t row_bytes,
                            std::vector<GatherJob>* out) {
  int64_t off = 0;
  for (int32_t c : counts) {
    if (c > 0) {
      GatherJob g = j;
      g.dst = j.dst + off * (int64_t)row_bytes;
      g.idx = j.idx ? j.idx + off : nullptr;
      g.idx2 = j.idx2 ? j.idx2 + off : nullptr;
      g.src = j.idx ? j.src : j.src + off * (int64_t)row_bytes;
      g.nrows = c;
      out->push_back(g);
    }
    off += c;
  }
  if (off < j.nrows) {  // rows beyond the listed messages (none for valid plans)
    GatherJob g = j;
    g.dst = j.dst + off * (int64_t)row_bytes;
    g.idx = j.idx ? j.idx + off : nullptr;
    g.idx2 = j.idx2 ? j.idx2 + off : nullptr;
    g.src = j.idx ? j.src : j.src + off * (int64_t)row_bytes;
    g.nrows = j.nrows - off;
    out->push_back(g);
  }
}

}  // namespace hx

// Host runtime of the C ABI: errors, device memory, topology handles,
// persistent requests (init / Start / Wait / backward), batches, the plain
// one-launch-per-member form, and the schedule tuner.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <numeric>
#include <sstream>
#include <string>
#include <utility>
#include <vector>

#include "common.h"
#include "internal.h"

namespace hx {

namespace {
thread_local std::string g_msg;
thread_local int g_hip = 0;
}  // namespace

int fail(int code, const char* fmt, ...) {
  char buf[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_msg = buf;
  return code;
}

int hip_fail(hipError_t e, const char* what, const char* file, int line) {
  g_hip = (int)e;
  char buf[1024];
  snprintf(buf, sizeof buf, "%s failed: %s (%s:%d)", what, hipGetErrorString(e), file, line);
  g_msg = buf;
  return e == hipErrorOutOfMemory ? HX_ERR_NOMEM : HX_ERR_HIP;
}

// Installed allocator (none: hipMalloc / hipFree).
namespace {
std::mutex g_alloc_mu;
hx_alloc_fn g_alloc_fn = nullptr;
hx_free_fn g_free_fn = nullptr;
void* g_alloc_ctx = nullptr;
}  // namespace

void DevMem::release() {
  if (p && owned) {
    if (free_fn) {
      // the caller's allocator may hand the block out again at once: wait
      // until no kernel still uses it, as hipFree does
      (void)hipDeviceSynchronize();
      free_fn(p, free_ctx);
    } else {
      (void)hipFree(p);
    }
  }
  p = nullptr;
  bytes = 0;
  free_fn = nullptr;
  free_ctx = nullptr;
  owned = true;
}

int DevMem::alloc(size_t nbytes, hipStream_t stream) {
  release();
  if (nbytes == 0) return HX_SUCCESS;
  hx_alloc_fn af;
  hx_free_fn ff;
  void* ctx;
  {
    std::lock_guard<std::mutex> lk(g_alloc_mu);
    af = g_alloc_fn;
    ff = g_free_fn;
    ctx = g_alloc_ctx;
  }
  if (af) {
    void* q = af(nbytes, (void*)stream, ctx);
    if (!q) return fail(HX_ERR_NOMEM, "the installed allocator failed to provide %zu bytes", nbytes);
    if (((uintptr_t)q & 15) != 0) {
      ff(q, ctx);
      return fail(HX_ERR_ARG, "the installed allocator returned a pointer that is not 16-byte aligned");
    }
    p = q;
    bytes = nbytes;
    free_fn = ff;
    free_ctx = ctx;
    return HX_SUCCESS;
  }
  hipError_t e = hipMalloc(&p, nbytes);
  if (e != hipSuccess) {
    p = nullptr;
    (void)hipGetLastError();
    g_hip = (int)e;
    return fail(HX_ERR_NOMEM, "hipMalloc(%zu) failed: %s", nbytes, hipGetErrorString(e));
  }
  bytes = nbytes;
  return HX_SUCCESS;
}

int upload(DevMem& dst, const void* host, size_t bytes) {
  HX_TRY(dst.alloc(bytes));
  if (bytes) HX_HIP(hipMemcpy(dst.p, host, bytes, hipMemcpyHostToDevice));
  return HX_SUCCESS;
}

int device_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    cached[dev] = v;
  }
  return cached[dev];
}

int device_lds_per_block() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 65536;
  if (cached[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
      v = 65536;
    cached[dev] = v;
  }
  return cached[dev];
}

// The default schedule of a phase.  The lines lie where sweeps over row sizes
// put them (4 to 256 bytes; 40 uneven requests of 76 to 131 MB a buffer, worlds
// of 509 to 4096 ranks and 18 to 600 MB a phase); us a call, the other side of
// a line first.
Sched default_sched(int kind, int row_bytes, const SchedFor& w) {
  constexpr int64_t kL2 = 4 << 20;  // one XCD's
  const int rb = std::max(row_bytes, 1);
  const bool one = rb == 4 || rb == 8;
  const bool pow2 = (rb & (rb - 1)) == 0;
  // streaming hints, for phases that move more than this: what a world's phase
  // reads was just written by the one before and is still in the 256 MB
  // Infinity Cache (copies of 400 MB 76 -> 63 without), a request's was not
  // (copies of 262 MB 58 -> 51 with; of 100 MB a call, cold 57 -> 38, and still
  // warm from the call before 27 -> 34)
  const bool streams = w.bytes >= (w.fresh ? (int64_t)1 << 30 : (int64_t)64 << 20);
  // a job's packed rows beyond the Infinity Cache, in short ascending runs
  const double packed = w.owned > 0 ? (double)w.source * (double)w.rows / (double)w.owned : 0;
  const bool scattered = packed > (double)(192 << 20) && 512 * w.runs > w.rows;
  // ascending runs that take every fourth of their source's rows, or more
  const bool dense = w.runs > 0 && 4.0 * (double)w.rows * (double)w.jobs >= (double)w.runs * (double)w.owned;
  Sched s;
  s.blocks_per_cu = kOneShotBpc;
  s.unroll = 4;
  if (kind == KIND_SEGSUM) {
    if (rb >= 64) {
      // the largest tile whose row pointers are staged in LDS; 1024 lanes: more
      // terms in flight per chunk, two each; a term is read once, so its loads
      // stream (128-B rows, 2.2 GB: 448 -> 422; 64 to 256 B: 5 to 12 %)
      s.tile_rows = std::min(kStageRows, std::max(64, (64 << 10) / rb));
      s.block_threads = 1024;
      s.unroll = 2;
      s.nontemporal = w.bytes >= (w.fresh ? (int64_t)256 << 20 : (int64_t)64 << 20) ? 1 : 0;
    } else if (rb == 8 && w.values == 2) {
      // two FP32 values: no row a lane; tiles whose pointers are staged in LDS
      // (above kStageRows every row is a chain of three loads: 40 uneven requests
      // 66 -> 21, 1024 ranks staged 129 -> 74, 4096 ranks staged 612 -> 388),
      // unless hardly a row has a term (1 M rows of 4000 terms 6.4, staged 9.2).
      // Rows of many terms fill the staging with few rows: their ranks' windows
      // where they fit (4096 ranks plain, 7 terms a row, 216 -> 135, in 512 rows
      // 265), else smaller tiles (100 ranks 34 -> 23, in 512 rows 29).  So do few
      // rows (16,384 rows of 3 terms in 512 rows 8.3, in 64 4.9).  A window's
      // workgroup has a lane a row: half as many where a rank has few (6000
      // requests of 100 rows of 8 terms 34 -> 23, 8000 of 30 rows of 20 59 -> 30;
      // of 200 rows and more both alike to 4 %).
      const bool many = w.terms > 6 * w.rows, none = 8 * w.terms <= w.rows;
      s.block_threads = 256;
      if (many && w.source <= kSegWinBytes) {
        s.lds_window = 1;
        s.tile_rows = 1024;
        s.block_threads = w.rows <= 128 * w.jobs ? 256 : 512;
      } else {
        s.tile_rows = many || w.rows < kStageRows * (int64_t)device_cus() ? 128 : none ? 1024 : kStageRows;
        s.unroll = 2;
      }
    } else if (one && w.source <= kL2) {
      // one row per lane, terms from LDS windows (1024 ranks staged backward,
      // FP32 189 -> 145, in tiles of 4096 rows 168: forwarders stage their
      // windows twice; 509 ranks plain, FP64 63 -> 48)
      s.pair_rows = 1;
      s.lds_window = 1;
      s.tile_rows = 8192;
      s.block_threads = 256;
    } else {
      // a persistent grid of 512-row tiles before: 8 B 143 -> 104, 12 B 101 ->
      // 75, 16 B 91 -> 77, 32 B 71 -> 65, 40 B 76 -> 70, 56 B 77 -> 64. Where
      // the terms are beyond the L2, tiles of 512 rows up to 40 B, half as many
      // terms in flight (12 B 139 -> 122, 16 B 123 -> 103, 20 B 119 -> 114,
      // 28 B 108 -> 101, 40 B 100 -> 94, 48 B 94 -> 90; two lanes a row of 32 B
      // fill the smaller tile: 92, 90). From the L2 12 B 155, in 512 rows 168.
      const bool far = w.source > kL2, two = rb == 32;
      // (hardly a term a row: 2.7 M rows of 40 B in tiles of 256 rows 46, of 512 34)
      const bool none = w.rows > 0 && 8 * w.terms <= w.rows;
      s.tile_rows = one || none || (far && rb <= 40 && !two) ? kStageRows : 256;
      s.block_threads = rb < (far && !two ? 20 : 40) ? 256 : 512;
      if (one || (far && rb <= 48)) s.unroll = 2;
    }
  } else if (w.identity) {
    // contiguous copies: 16 or 32 KiB a workgroup (one row per lane before:
    // 8-B rows, 153 MB: 40 -> 31)
    s.block_threads = streams ? 512 : 256;
    s.tile_rows = std::max(1, (streams ? 32 << 10 : 16 << 10) / rb);
    s.nontemporal = streams ? 1 : 0;
  } else if (w.phase == PH_PACK && rb >= 64 && rb <= 2048 && !w.fresh && 2 * w.rows <= w.owned) {
    // a request that packs half of its rows or fewer: the pull reads few of them
    // twice and walks no pointers (200 MB of rows packed in 6 messages, pushed and
    // pulled: three tenths of the rows 128 B 20.8 and 17.4, 400 B 46 and 20, a
    // tenth 12 and 7.4, 10.3 and 8.4, a fiftieth 8.8 and 3.9, 6.3 and 4.1; as many
    // as there are 80 B in 26 messages 17 and 23, three times as many of 60 MB
    // 128 B 37 and 44, 400 B 32 and 48; rows of 10 KB 8 and 12).  A world's packs
    // copy a caller's rows as they push them.
    s.tile_rows = std::max(16, (32 << 10) / rb);
    s.block_threads = 256;
  } else if (w.phase == PH_PACK && (rb >= 64 || (w.source > kL2 && 2 * w.rows >= w.owned && !scattered && !(dense && (one || w.rows <= w.owned))))) {
    // push: scattered full-line writes run as fast as scattered reads, and each
    // source row is read once; of shorter rows where the source is beyond the
    // L2, so that a pull's reads of parts of a line would go to memory (8 B
    // 103 -> 90, 16 B 70 -> 59, 24 B 68 -> 58, 40 B 67 -> 59; from a rank's own
    // rows, in the L2, 24 B 66 pulled and 85 pushed), and where at least half as
    // many rows are packed as the source has: a push walks every source row's
    // pointers.  4 M rows in 26 ascending messages, pulled and pushed: half of
    // the rows 8 B 38 and 27, 16 B 43 and 28, 24 B 49 and 44, 40 B 58 and 54; a
    // quarter 8 B 21 and 25, 24 B 27 and 40, 40 B 33 and 43; the surface of a
    // cube of 160 rows a side 8 B 7 and 24, 24 B 8 and 36.  Nor from messages
    // that take every fourth row or more, which a pull reads as whole lines (half
    // of the rows in two messages 8 B 16 and 26, 16 B 26 and 28; 1.2 M rows of 8 B
    // eight times in 26 messages 36 and 69; not longer rows read several times, 2 M
    // of 16 B thrice in 6 messages 36 and 24).  Nor from lists in no
    // order where what is packed is beyond the Infinity Cache: a push's writes of
    // parts of a line then go to memory one by one (12 M rows in runs of 64
    // ascending ones, 24 B, 274 MB, 295 and 378, of 512 294 and 303, of 4096 287
    // and 228; 40 B, 457 MB, 384 and 574, 442, 318; 16 B, 183 MB, 257 and 245).
    // Its writes merge in the
    // L2: no streaming hints (24 B 58, 152 with)
    s.push_pack = 1;
    // (400-B rows in tiles of 81 rows 181, of 40 155; where few of the rows are
    // packed the walk is what counts: a 64th of 1 M rows of 256 B in tiles of 64
    // rows 29, of 512 11, an eighth 43 and 21)
    s.tile_rows = rb <= 48 || 4 * w.rows < w.owned ? kStageRows
                  : std::max(16, std::min(256, (rb <= 192 ? 32 << 10 : 16 << 10) / rb));
    // (12 B 126 -> 119, 20 B 111 -> 106; 24 B 88, 82; a request's 200 B 104 -> 86,
    // 400 B 88 -> 72, 800 B 86 -> 68, of 80 B packed four times 80,
    // 90, of 200 B eight times 53, 66; a world's of 400 B that copies them 606, 624)
    s.block_threads = pow2 || rb < 24 || (rb >= 64 && rb <= 2048 && !w.fresh && w.rows <= 3 * w.owned) ? 256 : 512;
  } else if (one && w.phase == PH_PACK && w.bytes >= (int64_t)256 << 20) {
    // 16-byte row groups per lane; a rank's own rows are hot in the L2: no
    // window (4096 ranks 200 -> 165)
    s.pair_rows = 1;
    s.nontemporal = 1;
    s.tile_rows = 4096;
    s.block_threads = 512;
  } else if (one && w.phase != PH_PACK && w.rows >= 1 << 23) {
    // row groups, the job's window (if it has one) staged once per (up to)
    // 16384-row tile while the tile's indices are in flight (redistribution and
    // unpack of 39 M rows 476 -> 460; of 9 M FP32 ones 76 -> 72, with 512 lanes
    // and twice the groups, which spill, 86)
    s.pair_rows = 1;
    s.lds_window = 1;
    s.tile_rows = 16384;
    s.block_threads = rb == 8 ? 512 : 256;
    if (rb == 4) s.unroll = 2;
  } else if (one) {
    // what windows hold is in the caches anyhow (4.7 M rows: 86 -> 66), and one
    // row per lane reads runs of consecutive rows as whole lines (27-point
    // world of 766,000 rows 17.3 -> 15.0 a step); one pass of the workgroup a tile
    s.tile_rows = 1024;
    s.block_threads = 256;
  } else {
    // (24-B rows, packs 73 -> 66, redistribution and unpack 160 -> 150; 12 B
    // 45 -> 42)
    s.tile_rows = rb <= 16 ? 2048 : rb <= 32 ? 512 : 256;
    s.block_threads = 512;
  }
  // few rows: smaller tiles, down to 4 KiB of output, until every CU has two
  // (a window would then be staged by every one of them)
  const int64_t cus = device_cus();
  int64_t want = 2 * cus;
  int least = std::max(16, (4 << 10) / rb);
  if (kind == KIND_SEGSUM) {
    if (s.pair_rows) least = s.block_threads;  // (one-value sums: a row a lane)
    else if (rb > 8 && rb <= 16) least = 64;       // (8700 rows of 12 B, 8 terms each: 341 rows 14, 64 6)
  }
  const int64_t walked = s.push_pack ? w.owned : w.rows;  // rows that the tiles cover
  // (a world's ranks are one job where none reads a window: 1280 rows of 320 ranks
  // in one tile of 8192 13.4, in five 4.7)
  const int64_t jobs = w.fresh && !s.lds_window ? 1 : w.jobs;
  if (walked > 0 && jobs < cus && s.tile_rows > least && walked / s.tile_rows < want) {
    int64_t staged = 0;  // terms of a tile at most
    if (kind == KIND_SEGSUM && rb >= 64 &&
        (w.terms <= 3 * w.rows ? rb <= 2048 : rb <= 1024 && w.rows * rb <= 16 << 20)) {
      // 512 lanes, and a tile for every CU with no more terms than it stages: 1024
      // lanes wait for each other twice a tile (8 MB of rows of 64, 128 and 400 B, a
      // term or less each, 10.7 -> 5.4, 10.4 -> 5.3, 9.9 -> 5.2; 256 B of three each
      // 13.9 -> 8.0; 4 MB of five each, 64 to 800 B, 0.6 of the time.  27 MB of 200 B
      // of 8 each, more than a tile of 327 rows stages, 72 -> 148, in 163 rows 70 and
      // 84; 1600 B of five each 42 and 50)
      s.block_threads = 512;
      want = cus;
      least = std::max(16, (1 << 10) / rb);
      staged = kStageEntries * 3 / 4;
    }
    while (s.tile_rows > least &&
           (walked / s.tile_rows < want || (staged > 0 && s.tile_rows * w.terms > staged * w.rows)))
      s.tile_rows = std::max(least, s.tile_rows / 2);
    s.lds_window = 0;
    if (!s.push_pack && kind == KIND_GATHER) {
      s.block_threads = 256;
      s.unroll = 1;
    }
  }
  return s;
}

Sched resolve_sched(const hx_sched* p, int kind, int row_bytes, const SchedFor& w) {
  Sched s = default_sched(kind, row_bytes, w);
  if (!p) return s;
  if (p->tile_rows > 0) s.tile_rows = p->tile_rows;
  if (p->block_threads > 0) s.block_threads = p->block_threads;
  if (p->blocks_per_cu > 0) s.blocks_per_cu = p->blocks_per_cu;
  s.nontemporal = p->nontemporal <= 0 ? 0 : (p->nontemporal >= 2 ? 2 : 1);
  s.per_neighbor = p->per_neighbor ? 1 : 0;
  if (p->unroll > 0) s.unroll = p->unroll <= 1 ? 1 : (p->unroll == 2 ? 2 : 4);
  if (p->push_pack == 1) s.push_pack = 1;
  else if (p->push_pack == 2) s.push_pack = 0;
  if (p->lds_window == 1) s.lds_window = 1;
  else if (p->lds_window == 2) s.lds_window = 0;
  if (p->pair_rows == 1) s.pair_rows = 1;
  else if (p->pair_rows == 2) s.pair_rows = 0;
  return s;
}

hx_sched to_public(const Sched& s) {
  hx_sched o;
  o.tile_rows = s.tile_rows;
  o.block_threads = s.block_threads;
  o.blocks_per_cu = s.blocks_per_cu;
  o.nontemporal = s.nontemporal;
  o.per_neighbor = s.per_neighbor;
  o.unroll = s.unroll;
  o.push_pack = s.push_pack ? 1 : 2;
  o.lds_window = s.lds_window ? 1 : 2;
  o.pair_rows = s.pair_rows ? 1 : 2;
  return o;
}

}  // namespace hx

using namespace hx;

// ===========================================================================
// Topology
// ===========================================================================
static int check_procs(int rank, int nranks, int n, const int* procs, const char* what) {
  if (n < 0) return fail(HX_ERR_ARG, "%s: negative neighbor count", what);
  if (n > 0 && !procs) return fail(HX_ERR_ARG, "%s: null neighbor list", what);
  std::vector<int> v(procs, procs + n);
  for (int p : v)
    if (p < 0 || p >= nranks || p == rank)
      return fail(HX_ERR_RANGE, "%s: neighbor %d out of range or self", what, p);
  std::sort(v.begin(), v.end());
  if (std::adjacent_find(v.begin(), v.end()) != v.end())
    return fail(HX_ERR_RANGE, "%s: duplicate neighbor", what);
  return HX_SUCCESS;
}

extern "C" int hx_topo_create(int rank, int nranks, int n_recvs, const int* recv_procs,
                              const int* recv_weights, int n_sends, const int* send_procs,
                              const int* send_weights, int reorder, hx_topo** out) {
  (void)recv_weights;
  (void)send_weights;
  if (!out) return fail(HX_ERR_ARG, "null out");
  *out = nullptr;
  if (nranks <= 0 || rank < 0 || rank >= nranks) return fail(HX_ERR_ARG, "bad rank/nranks");
  if (reorder != 0) return fail(HX_ERR_UNSUPPORTED, "reorder is not supported (ranks are fixed)");
  HX_TRY(check_procs(rank, nranks, n_recvs, recv_procs, "recv_procs"));
  HX_TRY(check_procs(rank, nranks, n_sends, send_procs, "send_procs"));
  auto* t = new (std::nothrow) hx_topo;
  if (!t) return fail(HX_ERR_NOMEM, "out of host memory");
  t->rank = rank;
  t->nranks = nranks;
  t->recv_procs.assign(recv_procs, recv_procs + n_recvs);
  t->send_procs.assign(send_procs, send_procs + n_sends);
  *out = t;
  return HX_SUCCESS;
}

extern "C" int hx_topo_free(hx_topo** t) {
  if (!t) return HX_SUCCESS;
  delete *t;
  *t = nullptr;
  return HX_SUCCESS;
}

// ===========================================================================
// Requests
// ===========================================================================
static int req_phase_jobs(const hx_req* r, int phase, const Sched& sc, std::vector<GatherJob>* g,
                          std::vector<SegSumJob>* s);

// Launch table of one phase from its jobs: the backward is a segmented sum;
// the pack is a push (scatter) or a pull (gather) by the schedule; the other
// phases are gathers.
int hx::build_phase_table(int phase, const Sched& sc, int dtype, int row_bytes, const std::vector<GatherJob>& g,
                          const std::vector<SegSumJob>& s, LaunchTable* t) {
  if (phase == PH_BWD) return build_segsum_table(s, dtype, row_bytes, sc, t);
  // (a request with completion counters packs in the pull form whatever the schedule)
  if (phase == PH_PACK && sc.push_pack && g.empty()) return build_scatter_table(s, dtype, row_bytes, sc, t);
  if (phase == PH_PACK && !g.empty() && !s.empty())
    return fail(HX_ERR_STATE, "pack jobs of both forms in one launch");
  return build_gather_table(g, dtype, row_bytes, sc, t, phase);
}

SchedFor hx::req_sched_for(const hx_req* r, int phase) {
  const int64_t rb = (int64_t)r->row_bytes;
  SchedFor w;
  w.phase = phase;
  w.jobs = 1;
  w.values = r->ncols;
  w.bytes = r->bytes[phase];
  switch (phase) {
    case PH_PACK: w.rows = r->E1; w.owned = r->n_local; w.runs = r->pack_runs; w.source = r->n_local * rb; break;
    case PH_REDIST: w.rows = r->E2; w.source = r->R1 * rb; break;
    case PH_UNPACK: w.rows = r->H; w.source = (r->R1 + r->R2) * rb; w.identity = r->unpack_identity; break;
    default: w.rows = r->n_local; w.terms = r->E1; w.source = r->E1 * rb; break;
  }
  return w;
}

static int build_req_tables(hx_req* r) {
  if (r->tables_built) return HX_SUCCESS;
  // Wait's two gathers are independent (both read the receive arena): one
  // launch where they are short against a launch's 6 us (one rank's 9,000 rows
  // each way: 4 and 5 us)
  const bool one_wait =
      !r->unpack_identity && r->E2 > 0 && r->H > 0 && (r->E2 + r->H) * (int64_t)r->row_bytes <= 16 << 20;
  LaunchTable lt[4];
  for (int ph = 0; ph < 4; ++ph) {
    std::vector<GatherJob> g;
    std::vector<SegSumJob> s;
    const int kind = ph == PH_BWD ? KIND_SEGSUM : KIND_GATHER;
    if (one_wait && ph == PH_REDIST) continue;
    SchedFor w = req_sched_for(r, ph);
    if (one_wait && ph == PH_UNPACK) {
      w.rows += r->E2;
      w.jobs = 2;
      w.bytes += r->bytes[PH_REDIST];
      w.source = std::max(w.source, r->R1 * (int64_t)r->row_bytes);
    }
    const Sched sc = default_sched(kind, (int)r->row_bytes, w);
    if (one_wait && ph == PH_UNPACK) HX_TRY(req_phase_jobs(r, PH_REDIST, sc, &g, &s));
    HX_TRY(req_phase_jobs(r, ph, sc, &g, &s));
    HX_TRY(build_phase_table(ph, sc, r->dtype, (int)r->row_bytes, g, s, &lt[ph]));
  }
  std::move(lt, lt + 4, r->lt);  // (all or none: a call that fails leaves the request as it was)
  r->tables_built = true;
  return HX_SUCCESS;
}

static int req_phase_jobs(const hx_req* r, int phase, const Sched& sc, std::vector<GatherJob>* g,
                          std::vector<SegSumJob>* s) {
  const size_t rb = r->row_bytes;
  const bool per_nbr = sc.per_neighbor != 0;
  switch (phase) {
    case PH_PACK: {
      if (r->ready.p) {
        // partition-ready pack: pull form, one job per message, each with its
        // message's completion counter
        auto* cnt = r->ready.as<unsigned long long>();
        int64_t off = 0;
        for (size_t m = 0; m < r->s1_counts.size(); ++m) {
          const int64_t c = r->s1_counts[m];
          if (c > 0) {
            GatherJob j{r->x, r->send.as<char>() + off * (int64_t)rb, r->s1_idx.as<int32_t>() + off, c, 0, r->n_local};
            j.ready = cnt + m;
            g->push_back(j);
          }
          off += c;
        }
        break;
      }
      if (sc.push_pack) {
        if (r->E1 > 0)
          s->push_back(SegSumJob{r->x, r->send.as<char>(), r->bt_ptr.as<int32_t>(), r->bt_perm.as<int32_t>(),
                                 r->n_local});
        break;
      }
      GatherJob j{r->x, r->send.as<char>(), r->s1_idx.as<int32_t>(), r->E1, 0, r->n_local};
      if (per_nbr) split_gather_by_counts(j, r->s1_counts, rb, g);
      else g->push_back(j);
      break;
    }
    case PH_REDIST: {
      GatherJob j{r->recv.as<char>(), r->send.as<char>() + r->E1 * (int64_t)rb, r->s2_src.as<int32_t>(),
                  r->E2, 0, r->R1};
      if (per_nbr) split_gather_by_counts(j, r->s2_counts, rb, g);
      else g->push_back(j);
      break;
    }
    case PH_UNPACK: {
      GatherJob j{r->recv.as<char>(), r->halo, r->unpack_identity ? nullptr : r->unpack_src.as<int32_t>(),
                  r->H, 0, r->R1 + r->R2};
      if (per_nbr && r->unpack_identity) split_gather_by_counts(j, r->r1_counts, rb, g);
      else g->push_back(j);
      break;
    }
    case PH_BWD: {
      if (r->g_x && (r->g_send || r->E1 == 0)) {
        SegSumJob jb{r->g_send, r->g_x, r->bt_ptr.as<int32_t>(), r->bt_perm.as<int32_t>(), r->n_local};
        jb.win_rows = r->E1;  // the terms are the request's own send-slot gradients
        s->push_back(jb);
      }
      break;
    }
    default:
      return fail(HX_ERR_ARG, "bad phase");
  }
  return HX_SUCCESS;
}

int hx::req_jobs(const hx_req* r, int phase, const Sched& sc, std::vector<GatherJob>* g,
                 std::vector<SegSumJob>* s) {
  return req_phase_jobs(r, phase, sc, g, s);
}

static int64_t count_distinct_host(const std::vector<int32_t>& idx, int64_t domain) {
  if (idx.empty() || domain <= 0) return 0;
  std::vector<uint8_t> seen((size_t)domain, 0);
  int64_t u = 0;
  for (int32_t v : idx)
    if (v >= 0 && v < domain && !seen[v]) { seen[v] = 1; ++u; }
  return u;
}

void hx::req_compute_bytes(hx_req* r) {
  const int64_t rb = (int64_t)r->row_bytes;
  r->bytes[PH_PACK] = (r->E1 + r->U_pack) * rb + 4 * r->E1;
  r->bytes[PH_REDIST] = (r->E2 + r->U_redist) * rb + 4 * r->E2;
  r->bytes[PH_UNPACK] = 2 * r->H * rb + (r->unpack_identity ? 0 : 4 * r->H);
  r->bytes[PH_BWD] = (r->E1 + r->n_local) * rb + 4 * (r->E1 + r->n_local + 1);
}

// Builds the transpose of the pack map (rows -> send slots, ascending slot)
// on the host for list-initialised requests.
static void host_transpose(const std::vector<int32_t>& idx, int64_t n_local, std::vector<int32_t>* ptr,
                           std::vector<int32_t>* perm) {
  ptr->assign((size_t)n_local + 1, 0);
  for (int32_t v : idx) (*ptr)[(size_t)v + 1]++;
  for (int64_t i = 0; i < n_local; ++i) (*ptr)[(size_t)i + 1] += (*ptr)[(size_t)i];
  std::vector<int32_t> fill(ptr->begin(), ptr->end() - 1);
  perm->assign(idx.size(), 0);
  for (size_t k = 0; k < idx.size(); ++k) (*perm)[(size_t)fill[(size_t)idx[k]]++] = (int32_t)k;
}

static int check_layout(int n, const int* counts, const int* displs, int64_t* total, const char* what) {
  if (n > 0 && !counts) return fail(HX_ERR_ARG, "%s: null counts", what);
  int64_t acc = 0;
  for (int i = 0; i < n; ++i) {
    if (counts[i] < 0) return fail(HX_ERR_ARG, "%s: negative count", what);
    if (displs && displs[i] != acc)
      return fail(HX_ERR_ARG, "%s: displacement %d of neighbor %d is not the packed prefix %lld", what,
                  displs[i], i, (long long)acc);
    acc += counts[i];
  }
  if (acc >= INT32_MAX) return fail(HX_ERR_UNSUPPORTED, "%s: more than 2^31 rows", what);
  *total = acc;
  return HX_SUCCESS;
}

extern "C" int hx_neighbor_alltoallv_init(const void* x_local, int64_t n_local, const int* sendcounts,
                                          const int* sdispls, const int* send_idx, void* halo,
                                          const int* recvcounts, const int* rdispls, hx_dtype dtype,
                                          int ncols, const hx_topo* topo, hx_req** out) {
  if (!out) return fail(HX_ERR_ARG, "null out");
  *out = nullptr;
  if (!topo) return fail(HX_ERR_ARG, "null topology");
  if (dtype != HX_F32 && dtype != HX_F64) return fail(HX_ERR_ARG, "bad dtype");
  if (ncols <= 0) return fail(HX_ERR_ARG, "ncols must be positive");
  if (n_local < 0) return fail(HX_ERR_ARG, "negative n_local");
  if (n_local >= INT32_MAX) return fail(HX_ERR_UNSUPPORTED, "n_local beyond 2^31 rows");
  int64_t E = 0, H = 0;
  HX_TRY(check_layout((int)topo->send_procs.size(), sendcounts, sdispls, &E, "send"));
  HX_TRY(check_layout((int)topo->recv_procs.size(), recvcounts, rdispls, &H, "recv"));
  if (E > 0 && !send_idx) return fail(HX_ERR_ARG, "null send_idx");
  if (E > 0 && !x_local) return fail(HX_ERR_ARG, "null x_local");
  if (H > 0 && !halo) return fail(HX_ERR_ARG, "null halo");
  for (int64_t k = 0; k < E; ++k)
    if (send_idx[k] < 0 || send_idx[k] >= n_local)
      return fail(HX_ERR_RANGE, "send_idx[%lld] = %d outside [0, %lld)", (long long)k, send_idx[k],
                  (long long)n_local);
  std::unique_ptr<hx_req> r(new (std::nothrow) hx_req);
  if (!r) return fail(HX_ERR_NOMEM, "out of host memory");
  r->dtype = dtype;
  r->ncols = ncols;
  r->row_bytes = (size_t)ncols * dtype_bytes(dtype);
  r->variant = HX_PLAIN;
  r->rank = topo->rank;
  r->n_local = n_local;
  r->E1 = E;
  r->E2 = 0;
  r->R1 = H;
  r->R2 = 0;
  r->H = H;
  r->x = static_cast<const char*>(x_local);
  r->halo = static_cast<char*>(halo);
  r->unpack_identity = true;
  std::vector<int32_t> idx(send_idx, send_idx + E);
  r->s1_counts.assign(sendcounts, sendcounts + topo->send_procs.size());
  r->r1_counts.assign(recvcounts, recvcounts + topo->recv_procs.size());
  std::vector<int32_t> ptr, perm;
  host_transpose(idx, n_local, &ptr, &perm);
  HX_TRY(upload_vec(r->s1_idx, idx));
  HX_TRY(upload_vec(r->bt_ptr, ptr));
  HX_TRY(upload_vec(r->bt_perm, perm));
  HX_TRY(r->send.alloc((size_t)E * r->row_bytes));
  HX_TRY(r->recv.alloc((size_t)H * r->row_bytes));
  r->pack_runs = E > 0 ? 1 : 0;
  for (int64_t k = 1; k < E; ++k) r->pack_runs += idx[(size_t)k] < idx[(size_t)k - 1] ? 1 : 0;
  r->U_pack = count_distinct_host(idx, n_local);
  r->U_redist = 0;
  req_compute_bytes(r.get());
  *out = r.release();
  return HX_SUCCESS;
}

int hx::req_usable(const hx_req* r) {
  if (r->pending) return fail(HX_ERR_STATE, "the collective init this request joined has not completed");
  return HX_SUCCESS;
}

extern "C" int hx_start(hx_req* r, void* stream) {
  if (!r) return fail(HX_ERR_ARG, "null request");
  HX_TRY(req_usable(r));
  if (r->active) return fail(HX_ERR_STATE, "request already active");
  HX_TRY(build_req_tables(r));
  HX_TRY(launch_table(r->lt[PH_PACK], (hipStream_t)stream));
  r->active = true;
  return HX_SUCCESS;
}

extern "C" int hx_wait(hx_req* r, void* stream) {
  if (!r) return fail(HX_ERR_ARG, "null request");
  HX_TRY(req_usable(r));
  if (!r->active) return HX_SUCCESS;
  HX_TRY(build_req_tables(r));
  HX_TRY(launch_table(r->lt[PH_REDIST], (hipStream_t)stream));  // (empty where the unpack's table holds both)
  HX_TRY(launch_table(r->lt[PH_UNPACK], (hipStream_t)stream));
  r->active = false;
  return HX_SUCCESS;
}

extern "C" int hx_req_arena(hx_req* r, int which, void** dev_ptr, int64_t* rows) {
  if (!r || !dev_ptr || !rows) return fail(HX_ERR_ARG, "null argument");
  HX_TRY(req_usable(r));
  if (which == HX_ARENA_SEND) {
    *dev_ptr = r->send.p;
    *rows = r->E1 + r->E2;
  } else if (which == HX_ARENA_RECV) {
    *dev_ptr = r->recv.p;
    *rows = r->R1 + r->R2;
  } else {
    return fail(HX_ERR_ARG, "bad arena id");
  }
  return HX_SUCCESS;
}

extern "C" int hx_req_enable_ready(hx_req* r, unsigned long long** dev_counters) {
  if (!r || !dev_counters) return fail(HX_ERR_ARG, "null argument");
  HX_TRY(req_usable(r));
  if (r->active) return fail(HX_ERR_STATE, "request active");
  if (!r->ready.p) {
    const size_t n = std::max<size_t>(r->s1_counts.size(), 1);
    HX_TRY(r->ready.alloc(n * sizeof(unsigned long long)));
    HX_HIP(hipMemset(r->ready.p, 0, n * sizeof(unsigned long long)));
    r->tables_built = false;  // the pack is rebuilt per message
  }
  *dev_counters = r->ready.as<unsigned long long>();
  return HX_SUCCESS;
}

extern "C" int hx_req_bind_grad(hx_req* r, const void* g_send, void* g_x) {
  if (!r) return fail(HX_ERR_ARG, "null request");
  HX_TRY(req_usable(r));
  if ((r->E1 > 0 && !g_send) || (r->n_local > 0 && !g_x)) return fail(HX_ERR_ARG, "null gradient buffer");
  const char* const old_send = std::exchange(r->g_send, static_cast<const char*>(g_send));
  char* const old_x = std::exchange(r->g_x, static_cast<char*>(g_x));
  LaunchTable t;
  std::vector<GatherJob> g;
  std::vector<SegSumJob> s;
  const Sched sc = default_sched(KIND_SEGSUM, (int)r->row_bytes, req_sched_for(r, PH_BWD));
  int rc = req_phase_jobs(r, PH_BWD, sc, &g, &s);
  if (rc == HX_SUCCESS) rc = build_segsum_table(s, r->dtype, (int)r->row_bytes, sc, &t);
  if (rc != HX_SUCCESS) {  // the request keeps its former gradients
    r->g_send = old_send;
    r->g_x = old_x;
    return rc;
  }
  static std::atomic<uint64_t> bind_counter{0};
  r->grad_gen = ++bind_counter;  // batches holding this member rebuild their backward
  r->lt[PH_BWD] = std::move(t);
  return HX_SUCCESS;
}

extern "C" int hx_backward(hx_req* r, void* stream) {
  if (!r) return fail(HX_ERR_ARG, "null request");
  HX_TRY(req_usable(r));
  if (!r->g_x && r->n_local > 0) return fail(HX_ERR_STATE, "no gradient buffers bound");
  return launch_table(r->lt[PH_BWD], (hipStream_t)stream);
}

extern "C" int hx_req_free(hx_req** r) {
  if (!r || !*r) return HX_SUCCESS;
  if ((*r)->active) return fail(HX_ERR_STATE, "request active: wait before freeing it");
  if ((*r)->batch_refs > 0) return fail(HX_ERR_STATE, "request is a member of %d batch(es): free them first",
                                        (*r)->batch_refs);
  if ((*r)->comm) (*r)->comm->slot[(*r)->rank].req = nullptr;  // the collective forgets it
  delete *r;
  *r = nullptr;
  return HX_SUCCESS;
}

// ===========================================================================
// Batches
// ===========================================================================
namespace {

std::string arch_name() {
  int dev = 0;
  hipDeviceProp_t p;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&p, dev) != hipSuccess) return "unknown";
  std::string s = p.gcnArchName;
  auto c = s.find(':');
  return c == std::string::npos ? s : s.substr(0, c);
}

int ilog2(int64_t v) {
  int l = 0;
  while (v > 1) { v >>= 1; ++l; }
  return l;
}

std::mutex g_cache_mu;

}  // namespace

int hx::batch_phase_jobs(const hx_batch* b, int phase, const Sched& sc, bool merged,
                         std::vector<std::vector<GatherJob>>* g, std::vector<std::vector<SegSumJob>>* s) {
  g->clear();
  s->clear();
  if (b->world) return world_phase_jobs(b, phase, sc, merged, g, s);
  for (hx_req* r : b->members) {
    std::vector<GatherJob> gj;
    std::vector<SegSumJob> sj;
    HX_TRY(req_phase_jobs(r, phase, sc, &gj, &sj));
    if (b->tuning)  // candidate launches of the tuner leave completion counters alone
      for (auto& j : gj) j.ready = nullptr;
    g->push_back(gj);
    s->push_back(sj);
  }
  return HX_SUCCESS;
}

// Batched launch table of a phase under a schedule (all members' jobs).
int hx::batch_build_table(const hx_batch* b, int phase, const Sched& sc, LaunchTable* t) {
  std::vector<std::vector<GatherJob>> g;
  std::vector<std::vector<SegSumJob>> s;
  HX_TRY(batch_phase_jobs(b, phase, sc, true, &g, &s));
  *t = LaunchTable();
  std::vector<GatherJob> ga;
  std::vector<SegSumJob> sa;
  for (auto& v : g) ga.insert(ga.end(), v.begin(), v.end());
  for (auto& v : s) sa.insert(sa.end(), v.begin(), v.end());
  return build_phase_table(phase, sc, b->dtype, (int)b->row_bytes, ga, sa, t);
}

SchedFor hx::batch_sched_for(const hx_batch* b, int phase) {
  SchedFor w;
  if (b->world) {
    // a rank's share: its own rows (3-step: its node's), arena or slots
    const int64_t rb = (int64_t)b->row_bytes, R = std::max(b->R, 1);
    w.jobs = b->R;
    w.bytes = b->bytes[phase];
    w.fresh = true;
    const int64_t node = b->variant == HX_LOCALITY_3STEP ? b->ppn : 1;
    switch (phase) {
      case PH_PACK: w.rows = b->E1_tot; w.owned = b->n; w.source = b->n / R * node * rb; break;
      case PH_REDIST: w.rows = b->E2_tot; w.source = b->R1_tot / R * rb; break;
      case PH_UNPACK: w.rows = b->H_tot; w.source = b->R2_tot / R * rb; w.identity = b->unpack_identity; break;
      default:
        w.rows = b->n;
        w.terms = b->unpack_identity || b->staged_bwd ? b->E1_tot : b->H_tot;
        // (the closed-form adjoint reads every rank's halo, as one job)
        if (!b->unpack_identity && !b->staged_bwd) w.jobs = 1;
        w.source = b->unpack_identity || b->staged_bwd ? b->E1_tot / R * rb : b->H_tot * rb;
        break;
    }
  } else {
    double bytes = 0, weighted = 0;
    for (const hx_req* r : b->members) {
      const SchedFor m = req_sched_for(r, phase);
      w.rows += m.rows;
      w.owned += m.owned;
      w.runs += m.runs;
      w.terms += m.terms;
      w.jobs += m.rows > 0 ? 1 : 0;
      w.bytes += m.bytes;
      w.identity = m.identity;
      bytes += (double)m.bytes;
      weighted += (double)m.bytes * (double)m.source;
    }
    w.source = bytes > 0 ? (int64_t)(weighted / bytes) : 0;
    for (const hx_req* r : b->members) w.identity = w.identity && r->unpack_identity;
  }
  w.phase = phase;
  w.values = b->ncols;
  return w;
}

// One launch per member: the plain form, with the library's default schedule.
int hx::batch_build_plain(hx_batch* b, int phase) {
  std::vector<std::vector<GatherJob>> g;
  std::vector<std::vector<SegSumJob>> s;
  const int kind = phase == PH_BWD ? KIND_SEGSUM : KIND_GATHER;
  const Sched sc = default_sched(kind, (int)b->row_bytes, batch_sched_for(b, phase));
  HX_TRY(batch_phase_jobs(b, phase, sc, false, &g, &s));
  const size_t nm = std::max(g.size(), s.size());
  std::vector<LaunchTable> t(nm);
  for (size_t m = 0; m < nm; ++m) {
    static const std::vector<GatherJob> no_g;
    static const std::vector<SegSumJob> no_s;
    HX_TRY(build_phase_table(phase, sc, b->dtype, (int)b->row_bytes, m < g.size() ? g[m] : no_g,
                             m < s.size() ? s[m] : no_s, &t[m]));
  }
  b->plain[phase] = std::move(t);
  b->plain_built[phase] = true;
  return HX_SUCCESS;
}

// Forwarder sums of a staged locality world (bound gradients), one job per
// forwarder: its terms are its own halo's rows and, mostly, its own stage-2
// slots (the window).  Runs on the backward phase's schedule.
static int build_fwd_sum_table(const hx_batch* b, const Sched& sc, LaunchTable* t) {
  *t = LaunchTable();
  if (!b->staged_bwd || !b->g_out) return HX_SUCCESS;
  std::vector<SegSumJob> fjs;
  for (int q = 0; q < b->R; ++q) {
    const int64_t k0 = b->r1_off[q];
    SegSumJob fj{b->g_in, b->g_r1.as<char>() + k0 * (int64_t)b->row_bytes, b->fwd_ptr.as<int32_t>() + k0,
                 b->fwd_idx.as<int32_t>(), b->r1_off[q + 1] - k0};
    fj.in2 = b->g_s2.as<char>();
    fj.split = (int32_t)b->H_tot;
    fj.win_lo = b->H_tot + b->s2_off[q];
    fj.win_rows = b->s2_off[q + 1] - b->s2_off[q];
    fj.out2 = b->g_send_all.as<char>();
    fj.idx2 = b->gidx_from1.as<int32_t>() + k0;
    fjs.push_back(fj);
  }
  return build_segsum_table(fjs, b->dtype, (int)b->row_bytes, sc, t, TAG_FWD_SUM);
}

// Gradient bindings of a member batch's requests (the backward tables
// hold their g_send / g_x pointers).
static std::vector<uint64_t> member_grad_gens(const hx_batch* b) {
  std::vector<uint64_t> v;
  v.reserve(b->members.size());
  for (const hx_req* r : b->members) v.push_back(r->grad_gen);
  return v;
}

// (Re)builds the batched tables for the current schedules.  Start, Wait and the
// backward launch them one by one.  A hipGraph of them costs about 15 us a
// launch whatever it holds, a kernel launched from its table 2.7 us, and the
// longest of the three steps has four: captured graphs were never the faster
// replay (27-point world of 512 ranks, Start + Wait: 45.2 us from graphs, 26.8 so).
// All of the tables are replaced, or none: a call that fails leaves the batch with
// those it had.
int hx::batch_prepare(hx_batch* b) {
  LaunchTable lt[4], fwd_sum;
  for (int ph = 0; ph < 4; ++ph) HX_TRY(batch_build_table(b, ph, b->sched[ph], &lt[ph]));
  HX_TRY(build_fwd_sum_table(b, b->sched[PH_BWD], &fwd_sum));
  std::move(lt, lt + 4, b->lt);
  b->lt_fwd_sum = std::move(fwd_sum);
  if (!b->world) b->bwd_gens_built = member_grad_gens(b);
  return HX_SUCCESS;
}

int hx::batch_run_start(hx_batch* b, hipStream_t s) {
  return launch_table(b->lt[PH_PACK], s, {sim_transfer(b), 0, 0});
}

int hx::batch_run_wait(hx_batch* b, hipStream_t s) {
  HX_TRY(launch_table(b->lt[PH_REDIST], s, {sim_transfer(b), 0, 0}));
  return launch_table(b->lt[PH_UNPACK], s);
}

// Whether a phase's kernels write each row to its receiver too (the staged
// backward: its forwarder sums).
static bool delivers(const hx_batch* b, int phase) {
  return sim_transfer(b) && (phase == PH_PACK || phase == PH_REDIST || (phase == PH_BWD && b->staged_bwd));
}

static std::string cache_key(const hx_batch* b, int phase, bool delivering) {
  std::ostringstream k;
  int64_t rows = 0;
  int njobs = 0;
  std::vector<std::vector<GatherJob>> g;
  std::vector<std::vector<SegSumJob>> s;
  Sched neutral;  // the shape key counts rows of the pull form, whatever the schedule
  if (batch_phase_jobs(b, phase, neutral, true, &g, &s) == HX_SUCCESS) {
    for (auto& v : g) for (auto& j : v) { rows += j.nrows; ++njobs; }
    for (auto& v : s) for (auto& j : v) { rows += j.nrows; ++njobs; }
  }
  k << arch_name() << "|p" << phase << "|t" << b->dtype << "|rb" << b->row_bytes << "|r" << ilog2(rows + 1)
    << "|j" << ilog2(njobs + 1) << "|w" << (b->world ? 1 : 0);
  if (b->world) k << "|v" << b->variant;  // 2-step and 3-step worlds differ in shape
  if (phase == PH_BWD && b->staged_bwd) k << "|staged";  // forwarder + owner sums, not the closed form
  if (delivering) k << "|deliver";  // other kernels, with twice the writes
  return k.str();
}

static const char* cache_path() { return std::getenv("HX_TUNE_CACHE"); }

static bool cache_lookup(const std::string& key, Sched* out) {
  const char* path = cache_path();
  if (!path) return false;
  std::lock_guard<std::mutex> lk(g_cache_mu);
  std::ifstream f(path);
  std::string line;
  bool found = false;
  while (std::getline(f, line)) {
    std::istringstream ls(line);
    std::string k;
    Sched s;
    if (!(ls >> k >> s.tile_rows >> s.block_threads >> s.blocks_per_cu >> s.nontemporal >> s.per_neighbor >>
          s.unroll >> s.push_pack))
      continue;
    if (!(ls >> s.lds_window)) s.lds_window = 0;  // lines written before the field existed
    if (!(ls >> s.pair_rows)) s.pair_rows = 0;
    if (k == key) { *out = s; found = true; }
  }
  return found;
}

// A phase's tuned schedule.  (Files written before deliveries had a key of
// their own hold one for the shape.)
static bool cache_lookup(const hx_batch* b, int phase, Sched* out) {
  if (!cache_path()) return false;
  if (delivers(b, phase) && cache_lookup(cache_key(b, phase, true), out)) return true;
  return cache_lookup(cache_key(b, phase, false), out);
}

static void cache_store(const std::string& key, const Sched& s) {
  const char* path = cache_path();
  if (!path) return;
  std::lock_guard<std::mutex> lk(g_cache_mu);
  std::ofstream f(path, std::ios::app);
  f << key << ' ' << s.tile_rows << ' ' << s.block_threads << ' ' << s.blocks_per_cu << ' ' << s.nontemporal
    << ' ' << s.per_neighbor << ' ' << s.unroll << ' ' << s.push_pack << ' ' << s.lds_window << ' ' << s.pair_rows
    << '\n';
}

// Members with pack completion counters need the pull form of the pack.
static bool batch_has_ready(const hx_batch* b) {
  for (const hx_req* r : b->members)
    if (r->ready.p) return true;
  return false;
}

int hx::batch_init_scheds(hx_batch* b, const hx_sched* sched) {
  for (int ph = 0; ph < 4; ++ph) {
    b->sched_from_cache[ph] = sched == nullptr;
    const int kind = ph == PH_BWD ? KIND_SEGSUM : KIND_GATHER;
    if (sched) {
      b->sched[ph] = resolve_sched(sched, kind, (int)b->row_bytes, batch_sched_for(b, ph));
    } else {
      Sched s;
      b->sched[ph] = cache_lookup(b, ph, &s) ? s : default_sched(kind, (int)b->row_bytes, batch_sched_for(b, ph));
    }
  }
  if (batch_has_ready(b)) b->sched[PH_PACK].push_pack = 0;
  return HX_SUCCESS;
}

extern "C" int hx_batch_init(hx_req* const* reqs, int n, const hx_sched* sched, hx_batch** out) {
  if (!out) return fail(HX_ERR_ARG, "null out");
  *out = nullptr;
  if (n <= 0 || !reqs) return fail(HX_ERR_ARG, "empty batch");
  for (int i = 0; i < n; ++i) {
    if (!reqs[i]) return fail(HX_ERR_ARG, "null member %d", i);
    HX_TRY(req_usable(reqs[i]));
    if (reqs[i]->dtype != reqs[0]->dtype || reqs[i]->ncols != reqs[0]->ncols)
      return fail(HX_ERR_ARG, "members differ in dtype or ncols");
  }
  std::unique_ptr<hx_batch> b(new (std::nothrow) hx_batch);
  if (!b) return fail(HX_ERR_NOMEM, "out of host memory");
  b->world = false;
  b->dtype = reqs[0]->dtype;
  b->ncols = reqs[0]->ncols;
  b->row_bytes = reqs[0]->row_bytes;
  b->members.assign(reqs, reqs + n);
  for (int ph = 0; ph < 4; ++ph) {
    b->bytes[ph] = 0;
    for (hx_req* r : b->members) b->bytes[ph] += r->bytes[ph];
  }
  HX_TRY(batch_init_scheds(b.get(), sched));
  HX_TRY(batch_prepare(b.get()));
  for (hx_req* r : b->members) ++r->batch_refs;  // released by hx_batch_free
  *out = b.release();
  return HX_SUCCESS;
}

extern "C" int hx_batch_set_sched(hx_batch* b, int phase, const hx_sched* sched) {
  if (!b || !sched) return fail(HX_ERR_ARG, "null argument");
  if (phase < 0 || phase > 3) return fail(HX_ERR_ARG, "bad phase %d", phase);
  if (b->active) return fail(HX_ERR_STATE, "batch is active");
  const int kind = phase == PH_BWD ? KIND_SEGSUM : KIND_GATHER;
  const Sched old = b->sched[phase];
  b->sched[phase] = resolve_sched(sched, kind, (int)b->row_bytes, batch_sched_for(b, phase));
  if (phase == PH_PACK && batch_has_ready(b)) b->sched[PH_PACK].push_pack = 0;
  const bool deliveries = b->wp_to.p != nullptr;
  const int rc = batch_prepare(b);
  if (rc != HX_SUCCESS) {
    b->sched[phase] = old;
    if (!deliveries) b->wp_to.release();
  } else {
    b->sched_from_cache[phase] = false;
  }
  return rc;
}

extern "C" int hx_batch_set_replay(hx_batch* b, int mode) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (mode != HX_REPLAY_GRAPH && mode != HX_REPLAY_DIRECT) return fail(HX_ERR_ARG, "bad replay mode %d", mode);
  b->replay = mode;
  return HX_SUCCESS;
}

extern "C" int hx_batch_get_replay(const hx_batch* b, int* mode) {
  if (!b || !mode) return fail(HX_ERR_ARG, "null argument");
  *mode = b->replay;
  return HX_SUCCESS;
}

extern "C" int hx_batch_start(hx_batch* b, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (b->active) return fail(HX_ERR_STATE, "batch already active");
  HX_TRY(batch_run_start(b, (hipStream_t)stream));
  b->active = true;
  return HX_SUCCESS;
}

extern "C" int hx_batch_wait(hx_batch* b, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (!b->active) return HX_SUCCESS;
  HX_TRY(batch_run_wait(b, (hipStream_t)stream));
  b->active = false;
  return HX_SUCCESS;
}

extern "C" int hx_batch_start_plain(hx_batch* b, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (b->active) return fail(HX_ERR_STATE, "batch already active");
  hipStream_t s = (hipStream_t)stream;
  if (!b->plain_built[PH_PACK]) HX_TRY(batch_build_plain(b, PH_PACK));
  for (auto& t : b->plain[PH_PACK]) HX_TRY(launch_table(t, s, {sim_transfer(b), 0, 0}));
  b->active = true;
  return HX_SUCCESS;
}

extern "C" int hx_batch_wait_plain(hx_batch* b, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (!b->active) return HX_SUCCESS;
  hipStream_t s = (hipStream_t)stream;
  if (!b->plain_built[PH_REDIST]) HX_TRY(batch_build_plain(b, PH_REDIST));
  if (!b->plain_built[PH_UNPACK]) HX_TRY(batch_build_plain(b, PH_UNPACK));
  for (auto& t : b->plain[PH_REDIST]) HX_TRY(launch_table(t, s, {sim_transfer(b), 0, 0}));
  for (auto& t : b->plain[PH_UNPACK]) HX_TRY(launch_table(t, s));
  b->active = false;
  return HX_SUCCESS;
}

// Tables of a world's backward for the gradients b names now.  The arenas do not
// depend on them and are kept once made.
static int bind_world_tables(hx_batch* b) {
  const int rbi = (int)b->row_bytes;
  const Sched gsc = default_sched(KIND_GATHER, rbi);
  auto arena = [&](DevMem& m, int64_t rows) { return m.p ? HX_SUCCESS : m.alloc((size_t)rows * b->row_bytes); };
  LaunchTable back, back_copy, back2;
  if (!b->unpack_identity && !b->staged_bwd) HX_TRY(world_adjoint(b));
  if (b->unpack_identity) {
    // plain world: halo gradients travel back to the senders' slots (the
    // simulated reverse transfer), then each rank sums its own slots
    HX_TRY(arena(b->g_send_all, b->E1_tot));
    std::vector<GatherJob> xb{GatherJob{b->g_in, b->g_send_all.as<char>(), b->gidx_to1.as<int32_t>(), b->E1_tot}};
    HX_TRY(build_gather_table(xb, b->dtype, rbi, gsc, &back));
    // the same from a caller's buffer, which the bound one gets a copy of
    HX_TRY(world_from_map(b));
    GatherJob cb{b->g_in, nullptr, nullptr, b->H_tot};
    cb.dst2 = b->g_send_all.as<char>();
    cb.idx2 = b->gidx_from1.as<int32_t>();
    SchedFor cw;
    cw.identity = cw.fresh = true;
    HX_TRY(build_gather_table({cb}, b->dtype, rbi, default_sched(KIND_GATHER, rbi, cw), &back_copy));
  } else if (b->staged_bwd) {
    // locality world, staged: forwarder sums read the halo gradients (own
    // terms) and the stage-2 send-slot gradients (split = H)
    HX_TRY(arena(b->g_s2, b->E2_tot));
    HX_TRY(arena(b->g_r1, b->R1_tot));
    HX_TRY(arena(b->g_send_all, b->E1_tot));
    std::vector<GatherJob> x2{GatherJob{b->g_in, b->g_s2.as<char>(), b->gidx_back2.as<int32_t>(), b->E2_tot}};
    HX_TRY(build_gather_table(x2, b->dtype, rbi, gsc, &back2));
    HX_TRY(world_from_map(b));
  }
  HX_TRY(batch_prepare(b));
  b->lt_back = std::move(back);
  b->lt_back_copy = std::move(back_copy);
  b->lt_back2 = std::move(back2);
  return HX_SUCCESS;
}

extern "C" int hx_batch_bind_grad(hx_batch* b, const void* g_in, void* g_out) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (!b->world) return fail(HX_ERR_ARG, "member batches use each member's hx_req_bind_grad");
  // (empty buffers may be null: a decomposition without halo entries, or without rows)
  if ((!g_in && b->H_tot > 0) || (!g_out && b->n > 0)) return fail(HX_ERR_ARG, "null gradient buffer");
  const bool first = !b->g_out;
  const char* const old_in = std::exchange(b->g_in, static_cast<const char*>(g_in));
  char* const old_out = std::exchange(b->g_out, static_cast<char*>(g_out));
  const Sched old = b->sched[PH_BWD];
  // the backward's shape (and so its tuning-cache key) exists only now
  Sched cached;
  if (b->sched_from_cache[PH_BWD] && cache_lookup(b, PH_BWD, &cached)) b->sched[PH_BWD] = cached;
  const int rc = bind_world_tables(b);
  if (rc != HX_SUCCESS) {  // the batch keeps its former gradients, or none
    b->g_in = old_in;
    b->g_out = old_out;
    b->sched[PH_BWD] = old;
    if (first)
      for (DevMem* m : {&b->g_send_all, &b->g_s2, &b->g_r1, &b->gidx_from1, &b->wb_ptr, &b->wb_idx}) m->release();
    return rc;
  }
  b->halo_cols.release();  // (the adjoint is built)
  b->plain_built[PH_BWD] = false;
  return HX_SUCCESS;
}

static bool overlap(const void* p, size_t n, const void* q, size_t m) {
  return (const char*)p < (const char*)q + m && (const char*)q < (const char*)p + n;
}
static bool overlap(const void* p, size_t n, const DevMem& m) { return overlap(p, n, m.p, m.bytes); }

// Backward of a batch.  Plain worlds: with the simulated transport the reverse
// transfer first, then the owner sums.  Staged locality worlds: [reverse
// stage-2 transfer], forwarder sums (with the simulated transport written to the
// send slots they travel back to), owner sums.  Others: the fixed-order sums.
static int run_backward(hx_batch* b, hipStream_t s, bool plain_form, int64_t g_in, int64_t g_out) {
  const bool sim = sim_transfer(b);
  const bool plain_world = b->world && b->unpack_identity;
  const size_t gb = (size_t)b->H_tot * b->row_bytes, xb = (size_t)b->n * b->row_bytes;
  if (g_in != 0) {
    if (plain_world && sim && (b->lt_back_copy.empty() || b->lt_back_copy.deliver) &&
        !overlap(b->g_in + g_in, gb, b->g_send_all))
      HX_TRY(launch_table(b->lt_back_copy, s, {true, g_in, 0}));
    else {
      HX_HIP(hipMemcpyAsync(const_cast<char*>(b->g_in), b->g_in + g_in, gb, hipMemcpyDeviceToDevice, s));
      g_in = 0;
    }
  }
  if (b->world && b->staged_bwd) {
    if (sim) HX_TRY(launch_table(b->lt_back2, s));
    HX_TRY(launch_table(b->lt_fwd_sum, s, {sim, 0, 0}));
  } else if (plain_world && sim && g_in == 0) {
    HX_TRY(launch_table(b->lt_back, s));
  }
  if (!plain_form) {
    // (the owner sums copy theirs out as they go; not over what they still read)
    char* const out = b->g_out + g_out;
    const bool fused = g_out == 0 || !(overlap(out, xb, b->g_send_all) || overlap(out, xb, b->g_in, gb));
    HX_TRY(launch_table(b->lt[PH_BWD], s, {false, 0, fused ? g_out : 0}));
    if (!fused) HX_HIP(hipMemcpyAsync(out, b->g_out, xb, hipMemcpyDeviceToDevice, s));
    return HX_SUCCESS;
  }
  for (auto& t : b->plain[PH_BWD]) HX_TRY(launch_table(t, s));
  return HX_SUCCESS;
}

// Member gradients bound (or rebound to other buffers) since the backward
// tables were built: rebuild the tables (batched and plain).
static int refresh_member_grads(hx_batch* b) {
  if (b->world || member_grad_gens(b) == b->bwd_gens_built) return HX_SUCCESS;
  b->plain_built[PH_BWD] = false;
  Sched cached;  // gradients bound after the batch was made: the backward's cache key changes
  if (b->sched_from_cache[PH_BWD] && cache_lookup(b, PH_BWD, &cached)) b->sched[PH_BWD] = cached;
  return batch_prepare(b);
}

extern "C" int hx_batch_backward(hx_batch* b, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (b->world && !b->g_out) return fail(HX_ERR_STATE, "no gradient buffers bound");
  HX_TRY(refresh_member_grads(b));
  return batch_run_backward(b, (hipStream_t)stream);
}

extern "C" int hx_batch_backward_plain(hx_batch* b, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (b->world && !b->g_out) return fail(HX_ERR_STATE, "no gradient buffers bound");
  HX_TRY(refresh_member_grads(b));
  if (!b->plain_built[PH_BWD]) HX_TRY(batch_build_plain(b, PH_BWD));
  return run_backward(b, (hipStream_t)stream, true, 0, 0);
}

int hx::batch_run_backward(hx_batch* b, hipStream_t s, int64_t g_in, int64_t g_out) {
  return run_backward(b, s, false, g_in, g_out);
}

// Bytes from a bound buffer to a caller's of as many bytes (null, or the bound
// one itself: 0).
static int beside(const void* given, const void* bound, size_t bytes, const char* what, int64_t* out) {
  *out = given ? (int64_t)((uintptr_t)given - (uintptr_t)bound) : 0;
  if (*out % 16 != 0) return fail(HX_ERR_ARG, "%s: not aligned as the bound buffer (modulo 16 bytes)", what);
  if (*out != 0 && overlap(given, bytes, bound, bytes))
    return fail(HX_ERR_ARG, "%s: overlaps the bound buffer", what);
  return HX_SUCCESS;
}

extern "C" int hx_batch_exchange(hx_batch* b, const void* x, void* halo, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (!b->world) return fail(HX_ERR_ARG, "not a world batch");
  if (b->active) return fail(HX_ERR_STATE, "batch already active");
  hipStream_t s = (hipStream_t)stream;
  int64_t dx = 0, dh = 0;
  const size_t xb = (size_t)b->n * b->row_bytes, hb = (size_t)b->H_tot * b->row_bytes;
  HX_TRY(beside(x, b->x_global, xb, "x_global", &dx));
  HX_TRY(beside(halo, b->halo_all, hb, "halo_all", &dh));
  // (a push pack copies the rows as it goes; not from an arena that it writes)
  if (dx != 0 && (b->lt[PH_PACK].empty() || b->lt[PH_PACK].kind != KIND_SCATTER || overlap(x, xb, b->send_all) ||
                  overlap(x, xb, b->recv_all))) {
    HX_HIP(hipMemcpyAsync(const_cast<char*>(b->x_global), x, xb, hipMemcpyDeviceToDevice, s));
    dx = 0;
  }
  HX_TRY(launch_table(b->lt[PH_PACK], s, {sim_transfer(b), dx, 0}));
  HX_TRY(launch_table(b->lt[PH_REDIST], s, {sim_transfer(b), 0, 0}));
  // (a contiguous unpack copies its rows as it goes; not over the arena it reads)
  const bool fused = b->lt[PH_UNPACK].identity != 0 && !overlap(halo, hb, b->recv_all);
  HX_TRY(launch_table(b->lt[PH_UNPACK], s, {false, 0, fused ? dh : 0}));
  if (dh != 0 && !fused) HX_HIP(hipMemcpyAsync(halo, b->halo_all, hb, hipMemcpyDeviceToDevice, s));
  return HX_SUCCESS;
}

extern "C" int hx_batch_adjoint(hx_batch* b, const void* g_in, void* g_out, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (!b->world) return fail(HX_ERR_ARG, "not a world batch");
  if (!b->g_out) return fail(HX_ERR_STATE, "no gradient buffers bound");
  int64_t di = 0, dout = 0;
  const size_t rb = b->row_bytes;
  HX_TRY(beside(g_in, b->g_in, (size_t)b->H_tot * rb, "g_in", &di));
  HX_TRY(beside(g_out, b->g_out, (size_t)b->n * rb, "g_out", &dout));
  return batch_run_backward(b, (hipStream_t)stream, di, dout);
}

// One phase's kernel on its own, launched directly from the same
// launch table Start, Wait and the backward launch (for per-kernel timing).
extern "C" int hx_batch_launch_phase(hx_batch* b, int phase, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (phase < 0 || phase > 3) return fail(HX_ERR_ARG, "bad phase %d", phase);
  if (b->active) return fail(HX_ERR_STATE, "batch active: call hx_batch_wait first");
  if (phase == PH_BWD) {
    if (b->world && !b->g_out) return fail(HX_ERR_STATE, "no gradient buffers bound");
    if (!b->world && member_grad_gens(b) != b->bwd_gens_built)
      return fail(HX_ERR_STATE, "gradients bound after the last backward: call hx_batch_backward once first");
  }
  if (phase == PH_BWD && b->world && b->staged_bwd)  // the staged backward's forwarder sums first
    HX_TRY(launch_table(b->lt_fwd_sum, (hipStream_t)stream));
  return launch_table(b->lt[phase], (hipStream_t)stream);
}

extern "C" int hx_batch_get_sched(const hx_batch* b, int phase, hx_sched* out) {
  if (!b || !out || phase < 0 || phase > 3) return fail(HX_ERR_ARG, "bad argument");
  *out = to_public(b->sched[phase]);
  return HX_SUCCESS;
}

extern "C" int hx_batch_bytes(const hx_batch* b, int phase, int64_t* bytes) {
  if (!b || !bytes || phase < 0 || phase > 3) return fail(HX_ERR_ARG, "bad argument");
  *bytes = b->bytes[phase];
  return HX_SUCCESS;
}

// ---------------------------------------------------------------------------
// Tuner: times candidate schedules for each phase on the batch's buffers.
// ---------------------------------------------------------------------------
// Average launch time of a table: `reps` back-to-back launches between two
// events (queued faster than they run, so host launch cost stays hidden),
// best of two trials after a warm-up launch.  o: as a step launches it.
static int time_table(const LaunchTable& t, hipStream_t s, const LaunchOpt& o, hipEvent_t e0, hipEvent_t e1, int reps,
                      float* best) {
  HX_TRY(launch_table(t, s, o));  // warm-up
  *best = 1e30f;
  for (int trial = 0; trial < 2; ++trial) {
    HX_HIP(hipEventRecord(e0, s));
    for (int i = 0; i < reps; ++i) HX_TRY(launch_table(t, s, o));
    HX_HIP(hipEventRecord(e1, s));
    HX_HIP(hipEventSynchronize(e1));
    float ms = 0;
    HX_HIP(hipEventElapsedTime(&ms, e0, e1));
    *best = std::min(*best, ms / reps);
    // short kernels: enough launches for about a millisecond per trial (at
    // most 50), so that clock noise stays below the 2 % a candidate must win by
    if (trial == 0 && *best * reps < 1.0f) reps = std::min(50, std::max(reps, (int)std::ceil(1.0f / *best)));
  }
  return HX_SUCCESS;
}

extern "C" int hx_batch_tune(hx_batch* b, void* stream) {
  if (!b) return fail(HX_ERR_ARG, "null batch");
  if (b->active) return fail(HX_ERR_STATE, "batch is active");
  hipStream_t s = (hipStream_t)stream;
  hipEvent_t e0, e1;
  HX_HIP(hipEventCreate(&e0));
  HX_HIP(hipEventCreate(&e1));
  const bool log = std::getenv("HX_TUNE_LOG") != nullptr;  // every candidate's time on stderr
  struct TuningFlag {
    hx_batch* b;
    ~TuningFlag() { b->tuning = false; }
  } tuning_flag{b};
  b->tuning = true;
  int rc = HX_SUCCESS;
  for (int ph = 0; ph < 4 && rc == HX_SUCCESS; ++ph) {
    if (b->lt[ph].empty()) continue;
    const int kind = ph == PH_BWD ? KIND_SEGSUM : KIND_GATHER;
    const int rb = (int)b->row_bytes;
    // tiles around 32 KiB of output (segmented sums: the largest staged tile)
    const int base = kind == KIND_SEGSUM ? std::min(kStageRows, std::max(64, (64 << 10) / rb))
                     : rb == 4 || rb == 8 ? 16384
                                          : std::min(8192, std::max(64, (32 << 10) / rb));
    Sched best = b->sched[ph];
    float best_ms = 1e30f;
    auto consider = [&](const Sched& c) {
      if (rc != HX_SUCCESS) return;
      LaunchTable t;
      rc = batch_build_table(b, ph, c, &t);
      if (rc != HX_SUCCESS) return;
      float ms = 0;
      rc = time_table(t, s, {ph != PH_BWD && delivers(b, ph), 0, 0}, e0, e1, 3, &ms);
      if (rc == HX_SUCCESS && ph == PH_BWD && b->staged_bwd) {  // forwarder sums share the schedule
        LaunchTable tf;
        float msf = 0;
        rc = build_fwd_sum_table(b, c, &tf);
        if (rc == HX_SUCCESS) rc = time_table(tf, s, {delivers(b, ph), 0, 0}, e0, e1, 3, &msf);
        ms += msf;
      }
      if (log)
        std::fprintf(stderr, "hx tune phase %d: tile %d bt %d bpc %d nt %d unroll %d push %d win %d pair %d: %.4f ms\n",
                     ph, c.tile_rows, c.block_threads, c.blocks_per_cu, c.nontemporal, c.unroll, c.push_pack,
                     c.lds_window, c.pair_rows, ms);
      if (rc == HX_SUCCESS && ms < best_ms * 0.98f) {
        best_ms = ms;
        best = c;
      }
    };
    consider(best);
    // seeds for gathers of 4- and 8-byte rows: 16-byte row groups per lane,
    // one-shot grids, with whole-job LDS windows (sources in a known window)
    // and without (measured best on the random-matrix exchange); the
    // stage-by-stage search below refines from the fastest
    if (ph != PH_BWD && (rb == 4 || rb == 8) && !(ph == PH_PACK && best.push_pack)) {
      for (int win : {1, 0})
        for (int bt : {256, 512})
          for (int nt : {0, 1}) {
            Sched c = best;
            c.pair_rows = 1;
            c.lds_window = win;
            c.tile_rows = win ? 16384 : 4096;
            c.block_threads = bt;
            c.blocks_per_cu = kOneShotBpc;
            c.unroll = 4;
            c.nontemporal = nt;
            c.per_neighbor = 0;
            c.push_pack = 0;
            consider(c);
          }
    }
    // seeds for segmented sums of rows of one value: one row per lane,
    // per-job LDS term windows or none, one-shot grids
    if (ph == PH_BWD && (rb == 4 || rb == 8) && (size_t)rb == dtype_bytes(b->dtype)) {
      for (int win : {1, 0})
        for (int bt : {256, 512})
          for (int u : {2, 4}) {
            Sched c = best;
            c.pair_rows = 1;
            c.lds_window = win;
            c.tile_rows = 16384;
            c.block_threads = bt;
            c.blocks_per_cu = kOneShotBpc;
            c.unroll = u;
            c.nontemporal = 0;
            c.per_neighbor = 0;
            consider(c);
          }
    }
    // stage 1: work per tile, rows in flight, pull vs push (pack), LDS
    // source windows and two rows per lane (gathers); stage 2: launch shape
    // (persistent or one-shot grid, workgroup size) and streaming hints;
    // stage 3: stage 1 again around the new launch shape; stage 4: rows in
    // flight x launch shape
    auto tile_stage = [&]() {
      const Sched s0 = best;
      for (int tf : {1, 2, 4, 8, 16, 32})
        for (int u : {1, 2, 4})
          for (int push : {0, 1})
            for (int win : {0, 1})
              for (int pair : {0, 1}) {
                if (push && (ph != PH_PACK || batch_has_ready(b))) continue;
                if (win && push) continue;
                // 16-byte row groups per lane: pull gathers of 4- or 8-byte rows;
                // segmented sums of rows of one value: one row per lane
                if (pair && ((b->row_bytes != 8 && b->row_bytes != 4) || push ||
                             (ph == PH_BWD && b->row_bytes != dtype_bytes(b->dtype))))
                  continue;
                Sched c = s0;
                c.tile_rows = std::max(16, base * tf / 8);
                c.unroll = u;
                c.push_pack = ph == PH_PACK ? push : s0.push_pack;
                c.lds_window = win;
                c.pair_rows = pair;
                c.per_neighbor = 0;
                consider(c);
              }
    };
    tile_stage();
    {
      const Sched s1 = best;
      for (int bpc : {2, 4, 8, kOneShotBpc})
        for (int bt : {256, 512, 1024})
          for (int nt : {0, 1})
            for (int flip : {0, 1}) {
              // (gathers: LDS windows again with each launch shape, where the
              // occupancy they allow depends on the workgroup size)
              if (bt == 1024 && ph == PH_PACK && s1.push_pack) continue;  // push pack: at most 512 lanes
              if (flip && (ph == PH_BWD || (ph == PH_PACK && s1.push_pack))) continue;
              Sched c = s1;
              c.lds_window = flip ? !s1.lds_window : s1.lds_window;
              c.blocks_per_cu = bpc;
              c.block_threads = bt;
              c.nontemporal = nt;
              consider(c);
            }
    }
    tile_stage();
    // stage 4: rows in flight and launch shape together around the chosen
    // tile (the stage-by-stage search can stop at a near tie between them)
    {
      const Sched s3 = best;
      for (int u : {1, 2, 4})
        for (int bpc : {2, 4, 8, kOneShotBpc})
          for (int bt : {256, 512, 1024}) {
            if (bt == 1024 && ph == PH_PACK && s3.push_pack) continue;  // push pack: at most 512 lanes
            Sched c = s3;
            c.unroll = u;
            c.blocks_per_cu = bpc;
            c.block_threads = bt;
            consider(c);
          }
    }
    // stage 5: one job per message (member batches, pull forms)
    if (!b->world && !(ph == PH_PACK && best.push_pack) && ph != PH_BWD) {
      Sched c = best;
      c.per_neighbor = 1;
      consider(c);
    }
    // stage 6: streaming loads for the LDS window staging of 4- and 8-byte
    // row gathers (a window is read once; it pays where the arena was not
    // just left in the caches by the previous phase)
    if (ph != PH_BWD && (rb == 4 || rb == 8) && best.pair_rows && best.lds_window && !(ph == PH_PACK && best.push_pack)) {
      Sched c = best;
      c.nontemporal = 2;
      consider(c);
    }
    if (rc == HX_SUCCESS) {
      b->sched[ph] = best;
      b->sched_from_cache[ph] = false;  // tuned here: kept when gradients are bound again
      cache_store(cache_key(b, ph, delivers(b, ph)), best);
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  HX_TRY(rc);
  b->tuning = false;  // the tables kept for Start/Wait signal their counters again
  return batch_prepare(b);
}

extern "C" int hx_batch_free(hx_batch** b) {
  if (!b || !*b) return HX_SUCCESS;
  for (hx_req* r : (*b)->members) --r->batch_refs;
  delete *b;
  *b = nullptr;
  return HX_SUCCESS;
}

// ===========================================================================
// Errors / version
// ===========================================================================
extern "C" const char* hx_error_string(int code) {
  switch (code) {
    case HX_SUCCESS: return "success";
    case HX_ERR_ARG: return "invalid argument";
    case HX_ERR_RANGE: return "index out of range";
    case HX_ERR_STATE: return "invalid request state";
    case HX_ERR_NOMEM: return "out of memory";
    case HX_ERR_UNSUPPORTED: return "unsupported";
    case HX_ERR_HIP: return "HIP runtime error";
    default: return "unknown error";
  }
}

extern "C" int hx_set_allocator(hx_alloc_fn alloc_fn, hx_free_fn free_fn, void* ctx) {
  if ((alloc_fn == nullptr) != (free_fn == nullptr))
    return fail(HX_ERR_ARG, "hx_set_allocator: give both functions or neither");
  std::lock_guard<std::mutex> lk(g_alloc_mu);
  g_alloc_fn = alloc_fn;
  g_free_fn = free_fn;
  g_alloc_ctx = alloc_fn ? ctx : nullptr;
  return HX_SUCCESS;
}

extern "C" int hx_last_hip_error(void) { return g_hip; }
extern "C" const char* hx_last_error_message(void) { return g_msg.c_str(); }
extern "C" const char* hx_version(void) { return "hx 0.1 gfx950"; }

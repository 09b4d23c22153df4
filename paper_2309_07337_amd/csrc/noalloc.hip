// Entry point that allocates nothing: the backward of a request with its job
// in the launch's arguments (for callers that cannot allocate device memory
// during the call).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "internal.h"

extern "C" int hx_backward_noalloc(hx_req* r, const void* g_send, void* g_x, void* stream) {
  if (!r) return hx::fail(HX_ERR_ARG, "null request");
  HX_TRY(hx::req_usable(r));
  if (r->E1 > 0 && !g_send) return hx::fail(HX_ERR_ARG, "null g_send");
  if (r->n_local > 0 && !g_x) return hx::fail(HX_ERR_ARG, "null g_x");
  if (r->n_local == 0) return HX_SUCCESS;
  // the job of hx_backward, with these buffers instead of the bound ones
  hx::SegSumJob job{static_cast<const char*>(g_send), static_cast<char*>(g_x), r->bt_ptr.as<int32_t>(),
                    r->bt_perm.as<int32_t>(), r->n_local};
  job.win_rows = r->E1;  // the terms are the request's own send-slot gradients
  // the limit is stated in tiles of at most 512 rows, whatever the schedule's are
  const int limit_rows = std::min(512, std::max(64, (64 << 10) / (int)r->row_bytes));
  const int64_t tiles = (r->n_local + limit_rows - 1) / limit_rows, max_tiles = (HX_NOALLOC_SCRATCH_BYTES - 512) / 8;
  if (tiles > max_tiles)
    return hx::fail(HX_ERR_UNSUPPORTED, "%lld tiles of %d rows exceed %lld", (long long)tiles, limit_rows,
                    (long long)max_tiles);
  return hx::launch_segsum_one(job, r->E1, r->dtype, (int)r->row_bytes,
                               hx::default_sched(hx::KIND_SEGSUM, (int)r->row_bytes, hx::req_sched_for(r, hx::PH_BWD)),
                               (hipStream_t)stream);
}

// Pull-form row gathers: pack (Start), redistribution pack and unpack (Wait),
// and the backward's simulated transfers; short rows also in 16-byte groups per lane
// (the *_vec symbols).  One kernel symbol per phase (same body), so
// profiles attribute time to each phase separately.
#include "move_launch.h"

namespace hx {
namespace kern {
namespace {

#define HX_GATHER_KERNEL(NAME)                                                                 \
  template <int VB, int NV, int LPR, int U, bool NT, bool X>                                   \
  __global__ void __launch_bounds__(1024)                                                      \
      NAME(const GatherJob* __restrict__ jobs, const int64_t* __restrict__ ts, int njobs,      \
           int64_t ntiles, int tile_rows, int nv_rt, int use_win) {                            \
    gather_body<VB, NV, LPR, U, NT, X>(jobs, ts, njobs, ntiles, tile_rows, nv_rt, use_win);    \
  }                                                                                            \
  template <int VB, int U, bool NT, bool X>                                                    \
  __global__ void __launch_bounds__(1024)                                                      \
      NAME##_flat(const GatherJob* __restrict__ jobs, const int64_t* __restrict__ ts, int njobs, \
                  int64_t ntiles, int tile_rows, int nv) {                                     \
    gather_flat_body<VB, U, NT, X>(jobs, ts, njobs, ntiles, tile_rows, nv);                    \
  }                                                                                            \
  template <int RB, int U, bool NT, bool GAS, bool X>                                          \
  __global__ void __launch_bounds__(1024)                                                      \
      NAME##_vec(const GatherJob* __restrict__ jobs, const int64_t* __restrict__ ts, int njobs, \
                 int64_t ntiles, int tile_rows, int stream_win) {                              \
    gather_vec_body<RB, U, NT, GAS, X>(jobs, ts, njobs, ntiles, tile_rows, stream_win);        \
  }                                                                                            \
  template <bool X>                                                                            \
  struct NAME##_vgo {                                                                          \
    template <int RB, int U, bool NT>                                                          \
    static void go(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {                                      \
      const int sw = t.sched.nontemporal >= 2 ? 1 : 0; /* streaming window staging */          \
      if (t.partial_win)                                                                       \
        hipLaunchKernelGGL((NAME##_vec<RB, U, NT, false, X>), dim3(t.grid), dim3(t.sched.block_threads), \
                           (unsigned)t.win_bytes, s, t.jobs.as<GatherJob>(),                   \
                           t.tile_start.as<int64_t>(), t.njobs, t.ntiles, t.sched.tile_rows, sw); \
      else                                                                                     \
        hipLaunchKernelGGL((NAME##_vec<RB, U, NT, true, X>), dim3(t.grid), dim3(t.sched.block_threads), \
                           (unsigned)t.win_bytes, s, t.jobs.as<GatherJob>(),                   \
                           t.tile_start.as<int64_t>(), t.njobs, t.ntiles, t.sched.tile_rows, sw); \
    }                                                                                          \
  };                                                                                           \
  template <bool X>                                                                            \
  struct NAME##_go {                                                                           \
    template <int VB, int U, bool NT>                                                          \
    static void flat(const LaunchTable& t, hipStream_t s, const LaunchOpt& o, int nv) {                            \
      hipLaunchKernelGGL((NAME##_flat<VB, U, NT, X>), dim3(t.grid), dim3(t.sched.block_threads), \
                         0, s, t.jobs.as<GatherJob>(), t.tile_start.as<int64_t>(), t.njobs,    \
                         t.ntiles, t.sched.tile_rows, nv);                                     \
    }                                                                                          \
    template <int VB, int NV, int LPR, int U, bool NT>                                         \
    static void go(const LaunchTable& t, hipStream_t s, const LaunchOpt& o, int nv) {                              \
      hipLaunchKernelGGL((NAME<VB, NV, LPR, U, NT, X>), dim3(t.grid), dim3(t.sched.block_threads), \
                         (unsigned)t.win_bytes, s, t.jobs.as<GatherJob>(),                     \
                         t.tile_start.as<int64_t>(), t.njobs, t.ntiles, t.sched.tile_rows, nv, \
                         t.win_bytes > 0 ? 1 : 0);                                             \
    }                                                                                          \
  };
HX_GATHER_KERNEL(k_pack)
HX_GATHER_KERNEL(k_redist)
HX_GATHER_KERNEL(k_unpack)
HX_GATHER_KERNEL(k_transfer)
#undef HX_GATHER_KERNEL

// Contiguous copies (the plain unpack; with deliveries, the caller's halo
// gradients on their way back).
template <int VB, bool NT>
__global__ void __launch_bounds__(1024)
    k_unpack_copy(const GatherJob* __restrict__ jobs, const int64_t* __restrict__ ts, int njobs, int64_t ntiles,
                  int tile_rows, int row_bytes, Beside also) {
  copy_body<VB, NT>(jobs, ts, njobs, ntiles, tile_rows, row_bytes, also);
}

template <int VB>
__global__ void __launch_bounds__(1024)
    k_transfer_copy(const GatherJob* __restrict__ jobs, const int64_t* __restrict__ ts, int njobs, int64_t ntiles,
                    int tile_rows, int nv, Beside also) {
  copy_deliver_body<VB, 4>(jobs, ts, njobs, ntiles, tile_rows, nv, also);
}

template <int VB>
void copy_launch(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  if (o.deliver) {
    hipLaunchKernelGGL(k_transfer_copy<VB>, dim3(t.grid), dim3(t.sched.block_threads), 0, s, t.jobs.as<GatherJob>(),
                       t.tile_start.as<int64_t>(), t.njobs, t.ntiles, t.sched.tile_rows, t.row_bytes / VB,
                       Beside{o.src, 0});
    return;
  }
  // (with a second copy, streaming: it is read later than the caches hold)
  auto* kernel = t.sched.nontemporal || o.dst != 0 ? k_unpack_copy<VB, true> : k_unpack_copy<VB, false>;
  hipLaunchKernelGGL(kernel, dim3(t.grid), dim3(t.sched.block_threads), 0, s, t.jobs.as<GatherJob>(),
                     t.tile_start.as<int64_t>(), t.njobs, t.ntiles, t.sched.tile_rows, t.row_bytes, Beside{0, o.dst});
}

// The simulated transfer is not tuned: one fixed variant per shape.
struct transfer_fixed {
  template <int VB, int NV, int LPR, int U, bool NT>
  static void go(const LaunchTable& t, hipStream_t s, const LaunchOpt& o, int nv) {
    k_transfer_go<false>::go<VB, NV, LPR, (NV > 0 ? 4 : 1), false>(t, s, o, nv);
  }
};

template <int VB>
void transfer_shape(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  const int nv = t.row_bytes / VB;
  if constexpr (VB == 16) {
    if (nv == 8) return transfer_fixed::go<16, 8, 8, 4, false>(t, s, o, nv);
    if (nv == 16) return transfer_fixed::go<16, 16, 16, 4, false>(t, s, o, nv);
    if (nv == 1) return transfer_fixed::go<16, 1, 1, 4, false>(t, s, o, nv);
  } else if constexpr (VB == 8) {
    if (nv == 1) return transfer_fixed::go<8, 1, 1, 4, false>(t, s, o, nv);
  } else {
    if (nv == 1) return transfer_fixed::go<4, 1, 1, 4, false>(t, s, o, nv);
  }
  if (nv <= kFlatMaxVec) return k_transfer_go<false>::flat<VB, 4, false>(t, s, o, nv);
  return transfer_fixed::go<VB, 0, 64, 1, false>(t, s, o, nv);
}

// Short rows, 16 bytes per lane (the table builder set t.vec16): rows of 4
// or 8 bytes, U groups per lane in {1, 2, 4} (more would spill registers).
template <class F, int RB>
void vec_by_unroll(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  const bool nt = t.sched.nontemporal != 0;
  switch (unroll_bucket(t.sched.unroll)) {
    case 1: nt ? F::template go<RB, 1, true>(t, s, o) : F::template go<RB, 1, false>(t, s, o); break;
    case 2: nt ? F::template go<RB, 2, true>(t, s, o) : F::template go<RB, 2, false>(t, s, o); break;
    default: nt ? F::template go<RB, 4, true>(t, s, o) : F::template go<RB, 4, false>(t, s, o); break;
  }
}

template <class F>
void vec_launch(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  if (t.row_bytes == 8) vec_by_unroll<F, 8>(t, s, o);
  else vec_by_unroll<F, 4>(t, s, o);
}

}  // namespace
}  // namespace kern

void launch_gather_kernels(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  using namespace kern;
  if (o.deliver && !t.identity) {  // the pack and the redistribution only
    const bool pack = t.tag == TAG_PACK;
    if (t.vec16) pack ? vec_launch<k_pack_vgo<true>>(t, s, o) : vec_launch<k_redist_vgo<true>>(t, s, o);
    else pack ? by_vec<k_pack_go<true>>(t, s, o) : by_vec<k_redist_go<true>>(t, s, o);
    return;
  }
  if (t.identity) {
    if (t.vec_bytes == 16) copy_launch<16>(t, s, o);
    else if (t.vec_bytes == 8) copy_launch<8>(t, s, o);
    else copy_launch<4>(t, s, o);
    return;
  }
  if (t.vec16) {
    switch (t.tag) {
      case TAG_PACK: vec_launch<k_pack_vgo<false>>(t, s, o); return;
      case TAG_REDIST: vec_launch<k_redist_vgo<false>>(t, s, o); return;
      case TAG_UNPACK: vec_launch<k_unpack_vgo<false>>(t, s, o); return;
      // (a transfer's sources are runs of consecutive rows, which one row a lane
      // reads as whole lines: FP32, 9.6 M rows 28 us, in 16-byte groups 37)
      default: break;
    }
  }
  switch (t.tag) {
    case TAG_PACK: by_vec<k_pack_go<false>>(t, s, o); break;
    case TAG_REDIST: by_vec<k_redist_go<false>>(t, s, o); break;
    case TAG_UNPACK: by_vec<k_unpack_go<false>>(t, s, o); break;
    default:
      if (t.vec_bytes == 16) transfer_shape<16>(t, s, o);
      else if (t.vec_bytes == 8) transfer_shape<8>(t, s, o);
      else transfer_shape<4>(t, s, o);
      break;
  }
}

}  // namespace hx

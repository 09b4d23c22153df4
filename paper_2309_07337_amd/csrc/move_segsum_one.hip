// Fixed-order segmented sums of one job given in the launch's arguments (the
// backward that allocates nothing): the bodies of move_segsum.hip without a
// launch table.
#include "move_launch.h"

namespace hx {
namespace kern {
namespace {

template <class T, int VB, int NV, int LPR, int U, bool NT>
__global__ void __launch_bounds__(1024)
    k_segsum_one(SegSumJob job, int64_t ntiles, int tile_rows, int nv_rt, int cap_terms) {
  segsum_body<T, VB, NV, LPR, U, NT, true, false>(&job, nullptr, nullptr, 1, ntiles, tile_rows, nv_rt, cap_terms, Beside{0, 0});
}
template <class T, int VB, int U, bool NT>
__global__ void __launch_bounds__(1024)
    k_segsum_one_flat(SegSumJob job, int64_t ntiles, int tile_rows, int nv, int cap_terms) {
  segsum_flat_body<T, VB, U, NT, true, false>(&job, nullptr, nullptr, 1, ntiles, tile_rows, nv, cap_terms, Beside{0, 0});
}
template <class T, int U, int D, bool NT>
__global__ void __launch_bounds__(1024) k_segsum_one_vec(SegSumJob job, int64_t ntiles, int tile_rows) {
  segsum_vec_body<T, U, D, NT, true, false>(&job, nullptr, 1, ntiles, tile_rows, Beside{0, 0});
}

template <class T>
struct one_go {
  template <int VB, int U, bool NT>
  static void flat(const LaunchTable& t, hipStream_t s, const LaunchOpt& o, int nv) {
    if constexpr ((size_t)VB >= sizeof(T))  // (others are excluded when the table is shaped)
      hipLaunchKernelGGL((k_segsum_one_flat<T, VB, U, NT>), dim3(t.grid), dim3(t.sched.block_threads),
                         (unsigned)t.val_bytes, s, *o.one, t.ntiles, t.sched.tile_rows, nv, t.val_bytes / (nv * VB));
  }
  template <int VB, int NV, int LPR, int U, bool NT>
  static void go(const LaunchTable& t, hipStream_t s, const LaunchOpt& o, int nv) {
    const int vb = NV > 0 ? t.val_bytes : 0;  // term buffer (fixed shapes only)
    if constexpr ((size_t)VB >= sizeof(T))
      hipLaunchKernelGGL((k_segsum_one<T, VB, NV, LPR, U, NT>), dim3(t.grid), dim3(t.sched.block_threads),
                         (unsigned)vb, s, *o.one, t.ntiles, t.sched.tile_rows, nv, vb / (NV > 0 ? NV * VB : 1));
  }
};

template <class T, bool NT>
void one_vec(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  auto* kernel = t.vec_depth > 4                       ? k_segsum_one_vec<T, 1, 16, NT>
                 : unroll_bucket(t.sched.unroll) == 1 ? k_segsum_one_vec<T, 1, 4, NT>
                                                      : k_segsum_one_vec<T, 2, 4, NT>;
  hipLaunchKernelGGL(kernel, dim3(t.grid), dim3(t.sched.block_threads), (unsigned)t.win_bytes, s, *o.one, t.ntiles,
                     t.sched.tile_rows);
}

template <class T>
void one_launch(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  if (!t.vec16) by_vec<one_go<T>>(t, s, o);
  else if (t.sched.nontemporal) one_vec<T, true>(t, s, o);
  else one_vec<T, false>(t, s, o);
}

}  // namespace
}  // namespace kern

void launch_segsum_one_kernels(const LaunchTable& t, hipStream_t s, const LaunchOpt& o) {
  if (t.dtype == HX_F32) kern::one_launch<float>(t, s, o);
  else kern::one_launch<double>(t, s, o);
}

}  // namespace hx

// All three scans of a backward pass in one launch, 16-bit data, head_dim 128 and 64, gfx950.
#include "la2_scan_half.h"

namespace la2 {
namespace {
using namespace bf16k;

// The first half of the workgroups are the twin's (dK, dV of a chain and chunk), the second half run the dQ scan on the first half of
// their waves; the others end at once (a barrier counts the waves that are left).  The two kinds need nothing from each other, and
// each alone is short of work for the unit it runs on: at head_dim 64 (56 KiB of LDS, four waves) both of a chain share a unit, at
// 128, where a twin takes all of a unit's registers, a chain takes two units.  The long ones start first.  Two workgroups with the same
// place in their halves read the same tiles from opposite ends of the chain, on the same XCD when the halves are multiples of eight.
// Bound by memory from about half a round of workgroups on (d 64, 128 chains of 2048: 59 us for ten tensor passes of 32 MiB, 5.7 TB/s),
// below by the twin's block loop: 0.85 us a block of 32 positions at d 64, 2.0 at d 128.  When it is used: joint_plan in la2_api.hip.
template <typename E, int D, int CACHE, bool RS>
__global__ __launch_bounds__(4 * D, 128 / D) void bwd_scans_half_kernel(ScanParams dq, ScanParams rev) {
  __shared__ union {
    HalfLds<E, D, true, 3, false, false> twin;
    HalfLds<E, D, false, 3, false, false> one;
  } lds;
  const int units = (int)gridDim.x / 2, wg = (int)blockIdx.x;
  if (wg < units)
    [&]() __attribute__((always_inline)) { half_scan<E, D, CACHE, true, true, 3, false, false, RS>(rev, wg, lds.twin); }();
  else if (threadIdx.x < 2 * D)
    [&]() __attribute__((always_inline)) { half_scan<E, D, CACHE, false, false, 3, false, false, false>(dq, wg - units, lds.one); }();
}

template <typename E, int D>
hipError_t launch(const ScanParams& dq, const ScanParams& rev, dim3 g, hipStream_t s) {
  const dim3 b(4 * D);
  if (rev.keep != 0) {
    if (rev.ragged_state != 0) hipLaunchKernelGGL((bwd_scans_half_kernel<E, D, 1, true>), g, b, 0, s, dq, rev);
    else                       hipLaunchKernelGGL((bwd_scans_half_kernel<E, D, 1, false>), g, b, 0, s, dq, rev);
  } else {
    if (rev.ragged_state != 0) hipLaunchKernelGGL((bwd_scans_half_kernel<E, D, 0, true>), g, b, 0, s, dq, rev);
    else                       hipLaunchKernelGGL((bwd_scans_half_kernel<E, D, 0, false>), g, b, 0, s, dq, rev);
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_bwd_scans_bf16(int dtype, int head_dim, const ScanParams& dq, const ScanParams& rev, hipStream_t s) {
  if (dq.ragged_state != 0 || dq.acc_states != nullptr || dq.rstd != nullptr) return hipErrorInvalidValue;
  if (rev.nscan != 2 || rev.y[1] != rev.z[0] || rev.z[1] != rev.y[0]) return hipErrorInvalidValue;
  const int64_t grid = 2 * (dq.wg_map != nullptr ? (int64_t)dq.wg_pairs * dq.heads : (int64_t)dq.batch * dq.heads * dq.nchunks);
  if (grid == 0 || dq.n == 0) return hipSuccess;
  if (grid * 4 * head_dim > 0xFFFFFFFFll) return hipErrorInvalidValue;   // work-items (joint_plan in la2_api.hip sends no such call here)
  const dim3 g((unsigned)grid);
  if (head_dim == 64) return dtype == kF16 ? launch<_Float16, 64>(dq, rev, g, s) : launch<__bf16, 64>(dq, rev, g, s);
  return dtype == kF16 ? launch<_Float16, 128>(dq, rev, g, s) : launch<__bf16, 128>(dq, rev, g, s);
}

}  // namespace la2

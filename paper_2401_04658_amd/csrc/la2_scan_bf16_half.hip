// Half-block 16-bit scan kernels for head_dim 128 and 64, gfx950: one scan a workgroup, or the two reverse scans of the backward
// pass (twin), or a forward scan that forms the reverse chunk states on the side.  The body is in la2_scan_half.h.
#include "la2_scan_half.h"

namespace la2 {
namespace {
using namespace bf16k;

template <typename E, int D, int CACHE, bool REV, bool TWIN, int NBUF, bool NORM = false, bool ACC = false, bool RS = false>
__global__ __launch_bounds__(((TWIN || ACC) ? 4 : 2) * D, ((TWIN || ACC) ? 1 : 2) * (128 / D))
void scan_bf16_half_kernel(ScanParams p) {
  __shared__ HalfLds<E, D, TWIN, NBUF, NORM, ACC> lds;
  [&]() __attribute__((always_inline)) { half_scan<E, D, CACHE, REV, TWIN, NBUF, NORM, ACC, RS>(p, (int)blockIdx.x, lds); }();
}

}  // namespace

namespace {
template <typename E, int D, int CACHE>
hipError_t launch_half(bool reverse, bool twin, const ScanParams& p, hipStream_t s) {
  if (reverse != twin) return hipErrorInvalidValue;   // a reverse launch is the twin, a forward launch one scan
  const int64_t grid = p.wg_map != nullptr ? (int64_t)p.wg_pairs * p.heads : (int64_t)p.batch * p.heads * p.nchunks;
  // Three tile buffers in every case.  More buffers (5 for a plain, 4 for a twin workgroup that has the
  // compute unit to itself) measured no faster: such launches are bound by the memory system, not by the
  // bytes a workgroup keeps in flight.
  const dim3 g((unsigned)grid), plain(2 * D), twice(4 * D);   // threads: one wave per 32 value features, or two such groups
  if constexpr ((CACHE & 2) == 0) {   // (forward scans alone have the others)
    if (reverse) {
      if (p.ragged_state != 0) hipLaunchKernelGGL((scan_bf16_half_kernel<E, D, CACHE, true, true, 3, false, false, true>), g, twice, 0, s, p);
      else                     hipLaunchKernelGGL((scan_bf16_half_kernel<E, D, CACHE, true, true, 3>), g, twice, 0, s, p);
      return hipGetLastError();
    }
    if (p.acc_states != nullptr) {
      if (p.ragged_state != 0) return hipErrorInvalidValue;   // the host pairs these only with forward scans that do not accumulate
      hipLaunchKernelGGL((scan_bf16_half_kernel<E, D, CACHE, false, false, 3, false, true>), g, twice, 0, s, p);
      return hipGetLastError();
    }
  }
  if (reverse || p.acc_states != nullptr) return hipErrorInvalidValue;
  if (p.ragged_state != 0) {
    if (p.rstd == nullptr) hipLaunchKernelGGL((scan_bf16_half_kernel<E, D, CACHE, false, false, 3, false, false, true>), g, plain, 0, s, p);
    else                   hipLaunchKernelGGL((scan_bf16_half_kernel<E, D, CACHE, false, false, 3, true, false, true>), g, plain, 0, s, p);
  } else if (p.rstd != nullptr) {
    hipLaunchKernelGGL((scan_bf16_half_kernel<E, D, CACHE, false, false, 3, true>), g, plain, 0, s, p);
  } else {
    hipLaunchKernelGGL((scan_bf16_half_kernel<E, D, CACHE, false, false, 3>), g, plain, 0, s, p);
  }
  return hipGetLastError();
}
template <typename E, int D>
hipError_t launch_half_of(bool reverse, bool twin, const ScanParams& p, hipStream_t s) {
  // (the host asks for ordinary stores only on plain forward scans whose tiles are not kept)
  if (p.plain != 0 && !reverse && p.acc_states == nullptr) return launch_half<E, D, 2>(reverse, twin, p, s);
  return p.keep != 0 ? launch_half<E, D, 1>(reverse, twin, p, s) : launch_half<E, D, 0>(reverse, twin, p, s);
}
template <typename E>
hipError_t launch_half_of(int head_dim, bool reverse, bool twin, const ScanParams& p, hipStream_t s) {
  return head_dim == 64 ? launch_half_of<E, 64>(reverse, twin, p, s) : launch_half_of<E, 128>(reverse, twin, p, s);
}
}  // namespace

hipError_t launch_scan_bf16_half(int dtype, int head_dim, bool reverse, bool twin, const ScanParams& p, hipStream_t s) {
  return dtype == kF16 ? launch_half_of<_Float16>(head_dim, reverse, twin, p, s)
                       : launch_half_of<__bf16>(head_dim, reverse, twin, p, s);
}

}  // namespace la2

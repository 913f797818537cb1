// Recurrent decode step (Sec. 3.2.1, recursive form): kv <- lambda kv + k^T v, o = q kv, gfx950.
//
// Memory bound: the fp32 state (d x d per (batch, head)) is read and written once; everything
// else is negligible.  One workgroup (or a few) per (batch, head); each thread streams float4 pieces of the
// state rows with all of its loads issued up front, then the partial q.kv sums of the row groups
// are reduced through LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "la2_internal.h"

namespace la2 {
namespace {

// threads of a workgroup: a multiple of the D / 4 threads that share a state row, 16 or 12 float4 pieces
// of state rows per thread
constexpr int threads_for(int d) { return d == 256 ? 1024 : d == 96 ? 192 : 256; }
constexpr int split_threads(int d, int cs) { return d == 256 && cs == 2 ? 512 : 256; }

// element i of a tensor of type DT (kF32, kBF16 or kF16) as fp32, and the store that goes with it
template <int DT>
__device__ __forceinline__ float load_elem(const void* p, int64_t i) {
  if (DT == kBF16) return (float)reinterpret_cast<const __bf16*>(p)[i];
  if (DT == kF16) return (float)reinterpret_cast<const _Float16*>(p)[i];
  return reinterpret_cast<const float*>(p)[i];
}
template <int DT>
__device__ __forceinline__ void store_elem(void* p, int64_t i, float x) {
  if (DT == kBF16) reinterpret_cast<__bf16*>(p)[i] = (__bf16)x;
  else if (DT == kF16) reinterpret_cast<_Float16*>(p)[i] = (_Float16)x;
  else reinterpret_cast<float*>(p)[i] = x;
}

// CS: workgroups that share a chain, each with D / CS of the state's columns (column_split).  A thread holds at most 16
// pieces of 16 bytes in flight: 32 of them (256 threads at halves of head_dim 256) take 158 registers and leave three waves per SIMD.
// STREAM: the state passes by the caches (loads non-temporal, stores non-temporal and written through): see stream_state.
// NORM: the output row is normalised (eq. (2) read as root-mean-square normalisation over the head's features:
// o <- o / sqrt(mean_j o_j^2 + eps)) before it is stored.
template <int D, int DT, bool NORM, bool STREAM, int CS = 1>
__global__ __launch_bounds__(CS == 1 ? threads_for(D) : split_threads(D, CS)) void decode_kernel(const void* q, const void* k, const void* v,
                                                          const float* lambda, float* kv, void* o, int heads,
                                                          float eps) {
  static_assert(CS == 1 || !NORM, "the norm of a row needs all of its columns");
  constexpr int kThreads = CS == 1 ? threads_for(D) : split_threads(D, CS);
  constexpr int DC = D / CS;            // state columns of this workgroup
  constexpr int TPR = DC / 4;           // threads per state row (float4 each)
  constexpr int RG = kThreads / TPR;    // rows in flight per sweep
  constexpr int ITER = D / RG;
  __shared__ float sq[D], sk[D], sv[DC];
  __shared__ float4 sacc[RG][TPR];

  const int tid = threadIdx.x;
  const int64_t chain = blockIdx.x / CS;
  const int c0 = DC * (int)(blockIdx.x % CS);   // first column
  const float lam = lambda[chain % heads];
  if (tid < D) {
    sq[tid] = load_elem<DT>(q, chain * D + tid);
    sk[tid] = load_elem<DT>(k, chain * D + tid);
    if (tid < DC) sv[tid] = load_elem<DT>(v, chain * D + c0 + tid);
  }
  const int cg = tid % TPR, rg = tid / TPR;
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  typedef __attribute__((ext_vector_type(4))) int i32x4;
  f32x4* state = reinterpret_cast<f32x4*>(kv + chain * (int64_t)(D * D) + c0);
  const __amdgpu_buffer_rsrc_t streamed = __builtin_amdgcn_make_buffer_rsrc(state, 0, (D * D - c0) * 4, 0x00027000);
  f32x4 s[ITER];
#pragma unroll
  for (int it = 0; it < ITER; it++) {
    const f32x4* const at = &state[(int64_t)(rg + RG * it) * (D / 4) + cg];
    s[it] = STREAM ? __builtin_nontemporal_load(at) : *at;
  }
  __syncthreads();
  const float4 v4 = *reinterpret_cast<const float4*>(&sv[4 * cg]);
  float4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int it = 0; it < ITER; it++) {
    const int i = rg + RG * it;
    const float ki = sk[i], qi = sq[i];
    float4 t;
    t.x = fmaf(lam, s[it].x, ki * v4.x);
    t.y = fmaf(lam, s[it].y, ki * v4.y);
    t.z = fmaf(lam, s[it].z, ki * v4.z);
    t.w = fmaf(lam, s[it].w, ki * v4.w);
    const f32x4 tv = {t.x, t.y, t.z, t.w};
    if (STREAM) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, tv), streamed, (i * (D / 4) + cg) * 16, 0, 18);   // nt, sc1
    else        __builtin_nontemporal_store(tv, &state[(int64_t)i * (D / 4) + cg]);   // (4-7 % faster than the default policy)
    acc.x = fmaf(qi, t.x, acc.x);
    acc.y = fmaf(qi, t.y, acc.y);
    acc.z = fmaf(qi, t.z, acc.z);
    acc.w = fmaf(qi, t.w, acc.w);
  }
  sacc[rg][cg] = acc;
  __syncthreads();
  float sum = 0.f;
  if (tid < DC) {
    const float* flat = reinterpret_cast<const float*>(sacc);
#pragma unroll
    for (int g = 0; g < RG; g++) sum += flat[g * DC + tid];
  }
  if (NORM) {   // sum of squares over the row: inside each wave by lane exchanges, across the waves through LDS
    constexpr int NWAVE = (D + 63) / 64;   // waves that hold row elements
    __shared__ float ssq[NWAVE];
    float s2 = sum * sum;                  // 0 for tid >= D
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) s2 += __shfl_xor(s2, m);
    if (tid < D && (tid & 63) == 0) ssq[tid >> 6] = s2;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < NWAVE; i++) tot += ssq[i];
    sum *= 1.f / sqrtf(tot * (1.f / (float)D) + eps);
  }
  if (tid < DC) store_elem<DT>(o, chain * D + c0 + tid, sum);
}

__global__ void state_copy_kernel(float* dst, const float* src, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src ? src[i] : 0.f;
}

}  // namespace

hipError_t launch_state_copy(float* dst, const float* src, int64_t count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(state_copy_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, dst, src, count);
  return hipGetLastError();
}

// Whether a decode step's states pass by the caches.  A state that the 256 MiB memory-side cache still holds when the next step
// comes is better left there; a model of several layers goes through all their states before it returns to the first one,
// and what does not fit costs more than a stream.  Decode step, head_dim 128, through the caches (stores nt) against streaming,
// us: states of 64, 128, 256 MiB, one state used again at once 22.5 23.4, 43 47, 82 91; three in turn 22.5 23.4, 44 47, 106 92;
// twelve in turn 29.7 23.4, 55 47, 106 91.  Eight tokens a launch: 256 MiB 93 103, 114 104, 114 103.  The line lies between 128
// MiB, where the caches win with one and with three states in turn, and 256, where they win with one alone; many layers in turn
// would stream from 64 MiB on, a few would lose 4 to 9 % there.  Head_dim 256, whose
// workgroup has a compute unit to itself and loads and stores by turns, gains nothing (three of 256 MiB in turn 105, 106).
bool stream_state(int64_t chains, int head_dim) {
  return head_dim != 256 && chains * head_dim * head_dim * (int64_t)sizeof(float) >= (int64_t)160 << 20;
}

namespace {
// Workgroups that share a chain's state, a part of its columns each (the columns are independent of each other; not with the
// norm).  On few chains the launch is one workgroup's latency, and at head_dim 256 the undivided workgroup of 1024 threads has
// a compute unit to itself.  Undivided against divided, us, three states in turn / 768 MiB of states, which no cache holds:
// head_dim 256, quarters, 16 chains 5.8 3.4 / 8.9 4.7, 64 9.0 7.2 / 11.9 9.4; halves, 128 13.5 11.1 / 17.0 16.4, 256 24.8 23.2 /
// 27.1 29.4, 512 48.5 48.7 / 54.6 54.9, so the line is at 128.  Head_dim 128, halves, 16 chains 2.8 2.5 / 3.9 3.3, 64 3.2 2.9 /
// 4.5 4.1, 128 3.9 3.6 / 5.8 5.4, 256 6.7 6.8; quarters are no faster there (16 chains 2.5, 128 3.6).
int column_split(int64_t chains, int head_dim) {
  if (head_dim == 256) return chains <= 64 ? 4 : chains <= 128 ? 2 : 1;
  return head_dim == 128 && chains <= 128 ? 2 : 1;
}
}  // namespace

hipError_t launch_decode(int batch, int heads, int head_dim, int dtype, const void* q, const void* k,
                         const void* v, const float* lambda, float* kv, void* o, bool norm, float eps,
                         hipStream_t s) {
  const int64_t chains = (int64_t)batch * heads;
  if (chains == 0) return hipSuccess;
  dim3 g((unsigned)chains);
  const bool stream = stream_state(chains, head_dim);
  const int cs = norm ? 1 : column_split(chains, head_dim);
#define LA2_LAUNCH_DECODE_S(D, DT, STREAM)                                                                              \
  do {                                                                                                                  \
    if (norm) hipLaunchKernelGGL((decode_kernel<D, DT, true, STREAM>), g, dim3(threads_for(D)), 0, s, q, k, v, lambda, \
                                 kv, o, heads, eps);                                                                    \
    else      hipLaunchKernelGGL((decode_kernel<D, DT, false, STREAM>), g, dim3(threads_for(D)), 0, s, q, k, v, lambda, \
                                 kv, o, heads, eps);                                                                    \
  } while (0)
#define LA2_LAUNCH_DECODE_C(D, DT, CS)                                                                                  \
  hipLaunchKernelGGL((decode_kernel<D, DT, false, false, CS>), dim3(CS * g.x), dim3(split_threads(D, CS)), 0, s, q, k, v, \
                     lambda, kv, o, heads, eps)
#define LA2_LAUNCH_DECODE(D, DT)                                               \
  do {                                                                         \
    if (D == 256 && cs == 4)      LA2_LAUNCH_DECODE_C(256, DT, 4);             \
    else if (D == 256 && cs == 2) LA2_LAUNCH_DECODE_C(256, DT, 2);             \
    else if (D == 128 && cs == 2) LA2_LAUNCH_DECODE_C(128, DT, 2);             \
    else if (D != 256 && stream)  LA2_LAUNCH_DECODE_S(D, DT, D != 256);        \
    else                          LA2_LAUNCH_DECODE_S(D, DT, false);           \
  } while (0)
#define LA2_LAUNCH_DECODE_D(D)                         \
  do {                                                 \
    if (dtype == kBF16) LA2_LAUNCH_DECODE(D, kBF16);   \
    else if (dtype == kF16) LA2_LAUNCH_DECODE(D, kF16); \
    else LA2_LAUNCH_DECODE(D, kF32);                   \
  } while (0)
  if (head_dim == 256) LA2_LAUNCH_DECODE_D(256);
  else if (head_dim == 128) LA2_LAUNCH_DECODE_D(128);
  else if (head_dim == 96) LA2_LAUNCH_DECODE_D(96);
  else LA2_LAUNCH_DECODE_D(64);
#undef LA2_LAUNCH_DECODE_D
#undef LA2_LAUNCH_DECODE
#undef LA2_LAUNCH_DECODE_S
#undef LA2_LAUNCH_DECODE_C
  return hipGetLastError();
}

}  // namespace la2

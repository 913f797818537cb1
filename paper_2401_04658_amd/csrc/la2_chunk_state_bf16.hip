// Chunk-state pre-pass of the sequence-chunked launches, gfx950: local state of every chunk (bf16 MFMA, same
// streaming as the scan kernels) and the scan that turns local states into chunk start states (fp32).
#include <algorithm>

#include "la2_bf16_common.h"

namespace la2 {
namespace {
using namespace bf16k;

// Local state of every chunk that has a successor: forward sum_c lambda^(C-1-c) y_c^T z_c over the
// chunk's positions c, reverse sum_c lambda^c y_c^T z_c.  Written fp32 row-major [dk][dv].  Same
// streaming and the same state-update step as the scan kernel, without X, scores or outputs.
//
// A launch has about one workgroup per compute unit (it exists because the chains alone cannot fill the
// device) and hardly any arithmetic, so its speed is the bytes a workgroup keeps in flight: NBUF tile
// buffers, the tiles of block it + NBUF - 1 stream in while block it is used.  Every block's loads are
// issued unconditionally (past the chunk's end as dummy loads of one cache line), so the count of
// outstanding loads is the same in every iteration and one s_waitcnt immediate serves.
// The loads carry no non-temporal hint at any size: the scan behind this launch reads the same tiles again.  (Forward +
// backward of the packed 65,536 positions, sequences of up to 8192, H 16, d 128, with the streaming stores of the scans: 968 us
// with the hint, 914 without; one chain of 65,536, H 16: 874 and 868.  Without those stores it lost at the latter: 867, 897.)
// Two waves per SIMD: 2 NT waves (8 at d = 128, 4 at d = 64); wave w owns value features 32 (w % NT) .. + 31 and
// the key-feature tiles of half w / NT of the state slice, so that one wave's LDS and MFMA latencies hide behind
// the other's instructions (a wave issues one instruction at a time).
template <typename E, int D, bool REV, int NBUF>
__device__ __forceinline__ void chunk_state(const ScanParams& p, const int wg, E (&sT)[NBUF][2][Cfg<D>::TILE]) {
  static_assert(NBUF >= 3 && NBUF <= 5, "the block loop below is unrolled for 3 to 5 buffers");
  using C = Cfg<D>;
  constexpr int NT = C::NT, TILE = C::TILE;
  constexpr int KT = NT / 2;   // key-feature tiles per wave
  using Loader = TileLoader<D, 2, kB, 2 * NT>;
  constexpr int NDMA = 2 * Loader::DMA_PER_WAVE;   // direct loads per wave and block
  constexpr int VM_YOUNGER = (NBUF - 2) * NDMA;    // loads younger than those of block it + 1 when it waits for them
  static_assert(VM_YOUNGER < 64, "vmcnt is a 6-bit counter");
  constexpr int WAIT_NEXT_TILES = (VM_YOUNGER & 15) | ((VM_YOUNGER >> 4) << 14) | 0x0F70;

  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, l32 = l & 31, hh = l >> 5;
  const int dvt = w % NT, kt0 = (w / NT) * KT;
  int bi, hi, chunk, slot_stride, chunk_tokens;
  int64_t slot;
  if (!place_workgroup(p, wg, bi, hi, chunk, slot, slot_stride, chunk_tokens)) return;
  int64_t base;
  int n;
  chain_extent(p, bi, hi, base, n);
  const float l2 = log2f(p.lambda[hi]);
  const int nblocks = (n + kB - 1) / kB;
  const int cb = chunk_tokens / kB;
  const int blk_lo = chunk * cb;
  const int blk_hi = min(blk_lo + cb, nblocks);
  const int nblk = blk_hi - blk_lo;
  // the chunk a scan of THIS chain passes last has no successor (a packed batch: chains of different lengths)
  if (REV ? (chunk == 0) : (blk_hi >= nblocks)) return;

  Loader loader(w, l, n, (uint32_t)p.stride_n);
  loader.g[0] = reinterpret_cast<const char*>(reinterpret_cast<const E*>(p.y[0]) + base);
  loader.g[1] = reinterpret_cast<const char*>(reinterpret_cast<const E*>(p.z[0]) + base);
  const LaneAddr<D> la(l);
  const UpdateDecay<REV> decay(l2, hh);
  f32x16 kv[KT];
#pragma unroll
  for (int t = 0; t < KT; t++) kv[t] = zero16();

  // loads of the chunk's block number `it` (real, or dummy when the chunk has no such block) into `buf`
  auto issue_block = [&](E (*buf)[TILE], int it) __attribute__((always_inline)) {
    uint32_t doff[Loader::DMA_PER_WAVE];
    loader.offsets(REV ? blk_hi - 1 - it : blk_lo + it, it < nblk, doff);
#pragma unroll
    for (int j = 0; j < NDMA; j++) loader.template issue_one<true>(buf, doff, j);   // the scan reads these tiles again
  };
  if (nblk <= 0) return;
#pragma unroll
  for (int j = 0; j < NBUF - 1; j++) issue_block(sT[j], j);
  __builtin_amdgcn_s_waitcnt(WAIT_NEXT_TILES);   // the first block's tiles
  loader.zero_tail(sT[0], REV ? blk_hi - 1 : blk_lo);
  lds_barrier();

  auto block_step = [&](auto cur_tag, int it) __attribute__((always_inline)) -> bool {
    constexpr int cur = decltype(cur_tag)::value;
    const bool has_next = it + 1 < nblk;
    const int nb = REV ? blk_hi - 2 - it : blk_lo + it + 1;
    issue_block(sT[(cur + NBUF - 1) % NBUF], it + NBUF - 1);   // that buffer was block it - 1's
    const E* tY = sT[cur][0];
    const E* tZ = sT[cur][1];
    ex8<E> zf[4], yt[KT][4];   // [16-row k-step of the block]
#pragma unroll
    for (int k = 0; k < 4; k++) {
      zf[k] = la.read_cols(tZ, 16 * k, dvt);
#pragma unroll
      for (int t = 0; t < KT; t++) yt[t][k] = la.read_cols(tY, 16 * k, kt0 + t);
    }
    __builtin_amdgcn_sched_barrier(0);
    // Only the state after the chunk's last block is wanted, so instead of decaying the running sum by
    // lambda^B per block, each block's contribution carries its whole decay up front: the block processed
    // `it`-th has nblk - 1 - it blocks after it (forward: later positions; reverse: earlier ones), which
    // saves a quarter of the loop's vector instructions.  Exponents are non-negative: no overflow, and what
    // underflows is what the running decay would have wiped out as well.
    const float blk_decay = uniform(exp2f(l2 * (float)(kB * (nblk - 1 - it))));
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const ex8<E> zd = decay.apply(zf[k], 16 * k, blk_decay);
#pragma unroll
      for (int t = 0; t < KT; t++) kv[t] = mfma(yt[t][k], zd, kv[t]);
    }
    if (has_next) {
      __builtin_amdgcn_s_waitcnt(WAIT_NEXT_TILES);
      loader.zero_tail(sT[(cur + 1) % NBUF], nb);
      lds_barrier();   // next tiles visible to all waves; this block's buffer free
    }
    return has_next;
  };
  for (int it = 0;; it += NBUF) {   // unrolled by the number of buffers: compile-time buffer index
    if (!block_step(std::integral_constant<int, 0>{}, it)) break;
    if (!block_step(std::integral_constant<int, 1>{}, it + 1)) break;
    if (!block_step(std::integral_constant<int, 2 % NBUF>{}, it + 2)) break;
    if (NBUF > 3 && !block_step(std::integral_constant<int, 3 % NBUF>{}, it + 3)) break;
    if (NBUF > 4 && !block_step(std::integral_constant<int, 4 % NBUF>{}, it + 4)) break;
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // drain the dummy loads before the LDS is given up

  float* gs = p.states + slot * (D * D);   // a chunk with a successor: its chain has state slots
#pragma unroll
  for (int t = 0; t < KT; t++)
#pragma unroll
    for (int v = 0; v < 16; v++) gs[state_index<D>(dvt, l32, hh, kt0 + t, v, false)] = kv[t][v];
}

template <typename E, int D, bool REV, int NBUF>
__global__ __launch_bounds__(128 * (D / 32), 1) void chunk_state_bf16_kernel(ScanParams p) {
  __shared__ __attribute__((aligned(1024))) E sT[NBUF][2][Cfg<D>::TILE];   // [Y, Z]
  chunk_state<E, D, REV, NBUF>(p, (int)blockIdx.x, sT);
}

// Both families of a backward pass's chunk states in one launch: the first half of the workgroups the forward ones, the second
// half the reverse ones.
template <typename E, int D, int NBUF>
__global__ __launch_bounds__(128 * (D / 32), 1) void chunk_state_pair_bf16_kernel(ScanParams fwd, ScanParams rev) {
  __shared__ __attribute__((aligned(1024))) E sT[NBUF][2][Cfg<D>::TILE];
  const int units = (int)gridDim.x / 2, wg = (int)blockIdx.x;
  if (wg < units) chunk_state<E, D, false, NBUF>(fwd, wg, sT);
  else            chunk_state<E, D, true, NBUF>(rev, wg - units, sT);
}

// In place: states[chain][j] (local state of chunk j) -> start state of chunk j.
//   forward: G_0 = 0, G_{j+1} = lambda^C G_j + L_j        reverse: G_last = 0, G_{j-1} = lambda^C G_j + L_j
// The chunk processed first starts from init (element e read at its transposed place if init_tr) or 0.
// The carried state decays by lambda^(chunk length): all chunks are chunk_tokens long except the last
// one of the sequence, which a reverse scan passes first.
// A thread owns four consecutive elements of the d x d state.  It fetches the local states of kScanMaxChunks chunks
// (independent loads, all in flight together), runs the recurrence on registers and goes on to the next ones; the
// launch sits between two kernels that wait for it, so its latency is what counts, not its bytes.  (One chunk at a time
// beyond the first 32 it paid a round trip to memory per chunk: 1 chain of 65,536 positions, d 128, 256 chunks, forward +
// backward 0.313 -> 0.173 ms.)
constexpr int kScanMaxChunks = 32;
// wg_map != nullptr (packed batch with a compact grid, see ScanParams): a "unit" is a sequence of long_list and a
// head; the chain's states are `heads` slots apart.
__global__ __launch_bounds__(256) void state_scan_kernel(float* states, const float* lambda, int heads, int nchunks, int chunk_tokens,
                                  int dd, int reverse, const float* init, int init_tr, int d, int n,
                                  const int32_t* cu_seqlens, const int4* wg_map, const int32_t* long_list) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const int dd4 = dd >> 2;
  const int per_chain = (dd4 + (int)blockDim.x - 1) / (int)blockDim.x;   // workgroups per chain
  const int unit = (int)(blockIdx.x / per_chain);
  const int e4 = (int)(blockIdx.x % per_chain) * (int)blockDim.x + (int)threadIdx.x;
  if (e4 >= dd4) return;
  int bi, hi;
  int64_t first_slot, stride;   // the chain's chunk-0 state slot, slots between its consecutive chunks
  if (wg_map != nullptr) {
    const int pair = long_list[unit / heads];
    if (pair < 0) return;
    const int4 m = wg_map[pair];
    bi = m.x;
    chunk_tokens = m.w;
    hi = unit % heads;
    first_slot = (int64_t)m.z * heads + hi;
    stride = heads;
  } else {
    bi = unit / heads;
    hi = unit % heads;
    first_slot = (int64_t)unit * nchunks;
    stride = 1;
  }
  const int chain = bi * heads + hi;
  if (cu_seqlens != nullptr) n = cu_seqlens[bi + 1] - cu_seqlens[bi];   // this sequence's length
  int nch = (n + chunk_tokens - 1) / chunk_tokens;   // chunks this chain really has (<= nchunks)
  // (a packed sequence longer than the launch was planned for is the caller's error; it must not reach past the
  // chain's slots.  With a pair map the sequence's slots were counted from this same length.)
  if (wg_map == nullptr) nch = min(nch, nchunks);
  nch = __builtin_amdgcn_readfirstlane(nch);   // one chain per workgroup: scalar comparisons below
  const float l2 = log2f(lambda[hi]);
  const float lamFull = exp2f(l2 * (float)chunk_tokens);
  const float lamLast = exp2f(l2 * (float)(n - (nch - 1) * chunk_tokens));
  f32x4* s = reinterpret_cast<f32x4*>(states + first_slot * dd) + e4;
  const int64_t step = stride * dd4;   // f32x4 elements between consecutive chunks' states
  f32x4 g = {0.f, 0.f, 0.f, 0.f};
  if (init != nullptr) {
    const float* gi = init + (int64_t)chain * dd;
    const int e = 4 * e4;   // d is a multiple of 4: the four elements share a row
    if (init_tr) {
#pragma unroll
      for (int i = 0; i < 4; i++) g[i] = gi[((e + i) % d) * d + e / d];
    } else {
      g = *reinterpret_cast<const f32x4*>(gi + e);
    }
  }
#pragma unroll 1
  for (int i0 = 0; i0 < nch; i0 += kScanMaxChunks) {
    f32x4 loc[kScanMaxChunks];
#pragma unroll
    for (int i = 0; i < kScanMaxChunks; i++) {
      const int j = reverse ? nch - 1 - (i0 + i) : i0 + i;
      if (i0 + i < nch - 1) loc[i] = s[(int64_t)j * step];   // the chunk processed last has no successor: not read
    }
    // All of them have arrived: a wait between the stores below would be one for the stores before it.  (left: opaque, so
    // that the comparisons are made again and not kept from above in scalar registers.)
#pragma unroll
    for (int i = 0; i < kScanMaxChunks; i++) asm volatile("" : "+v"(loc[i]));
    int left = nch - i0;
    asm("" : "+s"(left));
#pragma unroll
    for (int i = 0; i < kScanMaxChunks; i++) {
      if (i < left) {
        const int j = reverse ? nch - 1 - (i0 + i) : i0 + i;
        s[(int64_t)j * step] = g;
        g = (j == nch - 1 ? lamLast : lamFull) * g + loc[i];   // (behind the last chunk: not used)
      }
    }
  }
}

// Packed batch in sequence chunks: the (sequence, chunk) pairs for the compact launch grid, the longest pairs first.
// One workgroup walks the sequences 256 at a time with a running count of pairs and of state slots.
//   map[pair] = {sequence, chunk, first state slot of the sequence (-1: single chunk, no slots), positions per chunk}
// Entries past the last pair, up to npairs, get sequence -1.  A batch whose lengths sum to more than the host was
// told would need more entries than the map has, or more state slots than the workspace (nslots per head): such
// sequences are dropped (nothing is written past the end of either; they are not computed).
// long_list[i] = pair of chunk 0 of the i-th sequence with state slots (i < nlong), -1 past the last.
//
// Order: a launch of this grid ends with whichever compute unit finishes last, and workgroups start in grid order.
// With the pairs in the order of the sequences a whole chunk could start when everything else was nearly done; sorted
// by length, in kLengthClasses classes, the short pairs fill the gaps that the long ones leave.  Forward + backward,
// bf16, 65,536 positions, H 16, d 128, the same cut in the order of the sequences and sorted: 42 sequences of 65 to
// 8192 positions 1.14 -> 1.06 ms; 55 of up to 4096, uncut, 0.99 -> 0.88 ms.
//
// Cost: one workgroup between the call and its first scan, so latency: one sequence per thread and round, no division for a
// sequence that is not cut, and a batch of one round is counted once and placed from registers.  2, 42, 923 and 3000
// sequences: 3.7, 5.1, 6.4, 17 us (256 at a time, counted twice, 4.7, 6.2, 11.7, 31).
constexpr int kLengthClasses = 64;
__global__ __launch_bounds__(1024) void varlen_map_kernel(const int32_t* cu_seqlens, int batch, int chunk_tokens, int npairs,
                                                          int4* map, int nlong, int32_t* long_list, int nslots,
                                                          int even_chunks) {
  __shared__ int wave_sum[16][3];
  __shared__ int at[kLengthClasses];   // first pass: pairs of every class; second: where the class's next pair goes
  const int t = (int)threadIdx.x, l = t & 63, w = t >> 6, round = (int)blockDim.x, nw = round >> 6;
  if (t < kLengthClasses) at[t] = 0;
  // class of a pair of `len` positions, at most chunk_tokens: 0 the longest
  const float per_class = (float)(kLengthClasses - 1) / (float)chunk_tokens;
  auto class_of = [&](int len) {
    return kLengthClasses - 1 - min((int)((float)min(len, chunk_tokens) * per_class), kLengthClasses - 1);
  };
  int len = 0, nch = 0, piece = chunk_tokens;       // this thread's sequence: positions, chunks, positions of all but the last
  int first_slot = 0, place = 0;                    // ... its first state slot, its place in long_list
  bool fits = false;
  int base_pairs = 0, base_slots = 0, base_long = 0;   // of the rounds before
  auto count_round = [&](int b) __attribute__((always_inline)) {
    len = nch = 0;
    // (a sequence without positions keeps one pair: its workgroups pass a start state on where one is handed over)
    if (b < batch) {
      len = max(cu_seqlens[b + 1] - cu_seqlens[b], 0);
      nch = len <= chunk_tokens ? 1
            : even_chunks       ? even_chunk_count(len, chunk_tokens)
                                : (int)(((uint32_t)len + (uint32_t)chunk_tokens - 1u) / (uint32_t)chunk_tokens);
    }
    const int slots = nch > 1 ? nch : 0;
    int ip = nch, is = slots, il = slots ? 1 : 0;   // inclusive scan of the three counts
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int yp = __shfl_up(ip, off), ys = __shfl_up(is, off), yl = __shfl_up(il, off);
      if (l >= off) { ip += yp; is += ys; il += yl; }
    }
    if (l == 63) { wave_sum[w][0] = ip; wave_sum[w][1] = is; wave_sum[w][2] = il; }
    __syncthreads();
    ip += base_pairs;
    is += base_slots;
    il += base_long;
    for (int i = 0; i < nw; i++) {
      const int sp = wave_sum[i][0], ss = wave_sum[i][1], sl = wave_sum[i][2];
      if (i < w) { ip += sp; is += ss; il += sl; }
      base_pairs += sp; base_slots += ss; base_long += sl;
    }
    __syncthreads();
    first_slot = is - slots;
    place = il - 1;
    fits = b < batch && ip <= npairs && (nch <= 1 || is <= nslots);
    if (even_chunks && nch > 1) piece = even_chunk_length(len, nch);
  };
  __syncthreads();
  for (int b0 = 0; b0 < batch; b0 += round) {
    count_round(b0 + t);
    if (fits) {
      if (nch > 1) atomicAdd(&at[class_of(piece)], nch - 1);
      atomicAdd(&at[class_of(len - (nch - 1) * piece)], 1);
    }
  }
  __syncthreads();
  if (w == 0) {   // counts -> first places, one class per lane
    const int own = at[l];
    int sum = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(sum, off);
      if (l >= off) sum += y;
    }
    at[l] = sum - own;
    if (l == 63) wave_sum[0][0] = sum;
  }
  __syncthreads();
  const int used = wave_sum[0][0], all_long = base_long;   // pairs of the sequences that are computed; sequences with slots
  __syncthreads();
  base_pairs = base_slots = base_long = 0;
  for (int b0 = 0; b0 < batch; b0 += round) {
    if (batch > round) count_round(b0 + t);
    if (fits) {
      const int first = nch > 1 ? atomicAdd(&at[class_of(piece)], nch - 1) : 0;
      for (int j = 0; j < nch - 1; j++) map[first + j] = make_int4(b0 + t, j, first_slot, piece);
      map[atomicAdd(&at[class_of(len - (nch - 1) * piece)], 1)] = make_int4(b0 + t, nch - 1, nch > 1 ? first_slot : -1, nch > 1 ? piece : chunk_tokens);
      if (nch > 1 && place < nlong) long_list[place] = first;
    } else if (nch > 1 && place < nlong) {
      long_list[place] = -1;
    }
  }
  for (int i = all_long + t; i < nlong; i += round) long_list[i] = -1;
  for (int i = used + t; i < npairs; i += round) map[i] = make_int4(-1, 0, -1, 0);
}

}  // namespace

namespace {
template <typename E>
hipError_t launch_chunk_states(int head_dim, bool reverse, const ScanParams& p, hipStream_t s) {
  const int64_t grid = p.wg_map != nullptr ? (int64_t)p.wg_pairs * p.heads : (int64_t)p.batch * p.heads * p.nchunks;
  dim3 g((unsigned)grid);
  if (head_dim == 128) {
    if (reverse) hipLaunchKernelGGL((chunk_state_bf16_kernel<E, 128, true, 4>), g, dim3(512), 0, s, p);
    else         hipLaunchKernelGGL((chunk_state_bf16_kernel<E, 128, false, 4>), g, dim3(512), 0, s, p);
  } else {
    if (reverse) hipLaunchKernelGGL((chunk_state_bf16_kernel<E, 64, true, 4>), g, dim3(256), 0, s, p);
    else         hipLaunchKernelGGL((chunk_state_bf16_kernel<E, 64, false, 4>), g, dim3(256), 0, s, p);
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_chunk_states_bf16(int dtype, int head_dim, bool reverse, const ScanParams& p, hipStream_t s) {
  const int64_t grid = (int64_t)p.batch * p.heads * p.nchunks;
  if (grid == 0 || p.n == 0) return hipSuccess;
  return dtype == kF16 ? launch_chunk_states<_Float16>(head_dim, reverse, p, s)
                       : launch_chunk_states<__bf16>(head_dim, reverse, p, s);
}

hipError_t launch_chunk_state_pair_bf16(int dtype, int head_dim, const ScanParams& fwd, const ScanParams& rev, hipStream_t s) {
  const int64_t grid = 2 * (fwd.wg_map != nullptr ? (int64_t)fwd.wg_pairs * fwd.heads : (int64_t)fwd.batch * fwd.heads * fwd.nchunks);
  if (head_dim != 64) return hipErrorInvalidValue;
  if (grid == 0 || fwd.n == 0) return hipSuccess;
  if (grid * 256 > 0xFFFFFFFFll) return hipErrorInvalidValue;   // work-items (joint_plan in la2_api.hip sends no such call here)
  const dim3 g((unsigned)grid), b(256);
  if (dtype == kF16) hipLaunchKernelGGL((chunk_state_pair_bf16_kernel<_Float16, 64, 4>), g, b, 0, s, fwd, rev);
  else               hipLaunchKernelGGL((chunk_state_pair_bf16_kernel<__bf16, 64, 4>), g, b, 0, s, fwd, rev);
  return hipGetLastError();
}

hipError_t launch_state_scan(int head_dim, bool reverse, const ScanParams& p, hipStream_t s) {
  const int64_t units = p.wg_map != nullptr ? (int64_t)p.nlong * p.heads : (int64_t)p.batch * p.heads;
  if (units == 0 || p.n == 0) return hipSuccess;
  const int dd = head_dim * head_dim;
  dim3 g((unsigned)(units * ((dd / 4 + 255) / 256))), b(256);   // the host checked that this fits a grid
  hipLaunchKernelGGL(state_scan_kernel, g, b, 0, s, p.states, p.lambda, p.heads, p.nchunks, p.chunk_tokens, dd,
                     reverse ? 1 : 0, p.init[0], p.init_transposed & 1, head_dim, p.n, p.cu_seqlens, p.wg_map, p.long_list);
  return hipGetLastError();
}

hipError_t launch_varlen_map(const ScanParams& p, int4* map, int32_t* long_list, int64_t nslots, hipStream_t s) {
  if (p.wg_pairs <= 0) return hipSuccess;
  hipLaunchKernelGGL(varlen_map_kernel, dim3(1), dim3(p.batch <= 256 ? 256 : 1024), 0, s, p.cu_seqlens, p.batch, p.chunk_tokens, p.wg_pairs, map,
                     p.nlong, long_list, (int)std::min<int64_t>(nslots, 0x7FFFFFFF), p.even_chunks);
  return hipGetLastError();
}

}  // namespace la2

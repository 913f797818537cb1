// fp32 kernels for the decayed causal scan (Algorithm 1; both loops of Algorithm 2), gfx950.
//
// fp32 storage and fp32 sums, for callers that need the 1e-5 accuracy class, on the bf16 matrix instructions.  A float is
// the exact sum of three bf16 numbers hi, mid, lo (8 significand bits each, the second and the third the rounded
// remainders: at most 2^-8 and 2^-17 of it), so a product of two floats is nine bf16 products; mid lo, lo mid and lo lo,
// together at most 2^-24 of the product and of either sign (rms 2^-27.5), are left out.  Six v_mfma_f32_32x32x16_bf16 (32
// cycles each) contract what eight v_mfma_f32_32x32x2_f32 (64 cycles each) do, in fewer rounded additions.
//
// Range.  lo of a value below 2^-110 would fall out of bf16's range, so every operand is scaled by 2^16 before it is split:
// X, Y, and Z with its weights; the state then carries 2^32, the scores 2^32, an output 2^48, taken off before it is
// stored.  Subnormals are operands like any other (bf16 parts reach down to 2^-133, 2^-149 after scaling: exact).  What
// leaves the range at the other end (an operand of 2^111 or more, a state or score of 2^95, an output of 2^79; Inf and
// NaN) turns some output or state element infinite or NaN, whatever else it meets.  A workgroup looks for that (one
// v_maximum3 per two outputs) and, if it finds it, walks its chunk again on v_mfma_f32_32x32x2_f32: that walk's state, and
// its outputs from the first such block on, are what is kept.  Its tiles are fp32 in the place of the planes; it is written
// for registers, not for speed.
//
// Organisation: one workgroup walks the blocks (B = 32 positions) of one sequence chunk of one (batch, head) chain;
// wave w owns value features 32 w .. 32 w + 31 of the output and of the running state, whose slice stays in MFMA
// accumulator registers and is split into operands straight from there.  X and Y tiles are split once, by the thread
// that loads them, and sit in LDS as three bf16 planes each (the tile layout of the 16-bit kernels); a wave's own
// columns of Z go from global memory to its registers and are split there (no other wave needs them).  The masked
// score tile is the same for all waves: they compute it in 16 x 16 quarters (v_mfma_f32_16x16x32_bf16) and exchange it
// through LDS.
//
// One tile buffer: the next block's values are on their way to registers while a block is computed, and are split
// into the planes between the block's two barriers.  56 KiB (D = 128) or 32 KiB (D = 64) of LDS and 256 registers, so
// two (four) workgroups share a compute unit and one computes while the other splits and waits.
//
// What bounds it: issue.  Per wave and block 3,840 cycles of matrix pipe and about 930 vector instructions (the split is
// 5.5 per element: 64 elements of the state, 64 of the tiles; 58 for the scaling and the look at the outputs; the pipes
// share the issue, at full load both are half busy).  Against v_mfma_f32_32x32x2_f32 on tiles in fp32 (208 of 64 cycles, one
// workgroup per unit), forward + backward: batch 4, H 16, n 2048, d 128 0.856 -> 0.417 ms, batch 16, n 1024 1.20 -> 0.63;
// d 64, batch 4, n 2048 0.330 -> 0.200, batch 16, n 1024 0.57 -> 0.33 (without the scaling and the look 0.405, 0.60, 0.194,
// 0.31).  Relative error of the results (2-norm, N(0, 1) data, n 200) 2.5e-7 -> 2.0e-7 at d 128, 2.1e-7 -> 1.7e-7 at d 64.
//
// Feature order.  In the accumulator layout a lane holds rows 8 (v / 4) + 4 hh + v % 4 of a state tile, so the eight
// elements of a k-step would not be the eight consecutive features of an X row fragment.  The transposing reads of Y
// take the columns with bits 2 and 3 of the index exchanged (the lanes pass the addresses of the 8-byte pieces in that
// order); state register (t, v) then is key feature 32 t + 16 (v / 8) + 8 hh + v % 8 and a k-step's elements are
// features 16 ks + 8 hh .. + 7.
#include "la2_bf16_common.h"

namespace la2 {
namespace {
using namespace bf16k;

constexpr int kBF = 32;   // block size (positions per block)
constexpr float kUp = 65536.f;   // 2^16: what an operand is scaled by before it is split
typedef ex8<__bf16> b8;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {   // contracts two indices, one per wave half
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// the three bf16 parts of a pair of floats, packed (low half: the first)
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  auto pk = [](float x, float y) __attribute__((always_inline)) {
    const f32x2 v = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  };
  hi = pk(a, b);
  a -= __uint_as_float(hi << 16);
  b -= __uint_as_float(hi & 0xFFFF0000u);
  mid = pk(a, b);
  a -= __uint_as_float(mid << 16);
  b -= __uint_as_float(mid & 0xFFFF0000u);
  lo = pk(a, b);
}

struct Parts {   // an operand of eight floats: its parts, the largest first
  b8 p[3];
};
__device__ __forceinline__ Parts split8(const float (&x)[8]) {
  union { uint32_t u[4]; b8 v; } r[3];
#pragma unroll
  for (int i = 0; i < 4; i++) split2(x[2 * i], x[2 * i + 1], r[0].u[i], r[1].u[i], r[2].u[i]);
  return Parts{{r[0].v, r[1].v, r[2].v}};
}

// hi lo, lo hi, mid mid (at most 2^-16 of the whole), hi mid, mid hi, hi hi, in this order
template <typename Acc, typename F>
__device__ __forceinline__ Acc six(const Parts& a, const Parts& b, Acc c, F f) {
  c = f(a.p[0], b.p[2], c);
  c = f(a.p[2], b.p[0], c);
  c = f(a.p[1], b.p[1], c);
  c = f(a.p[0], b.p[1], c);
  c = f(a.p[1], b.p[0], c);
  return f(a.p[0], b.p[0], c);
}
__device__ __forceinline__ f32x16 mul32(const Parts& a, const Parts& b, f32x16 c) {
  return six(a, b, c, [](b8 x, b8 y, f32x16 z) __attribute__((always_inline)) { return mfma(x, y, z); });
}
__device__ __forceinline__ f32x4 mul16(const Parts& a, const Parts& b, f32x4 c) {
  return six(a, b, c, [](b8 x, b8 y, f32x4 z) __attribute__((always_inline)) { return mfma16(x, y, z); });
}

// The same split in eight steps of five or six vector instructions, each closed by pins: side work for the shadow of
// six MFMAs (step(i) beside the i-th).
struct Splitter {
  float x[8];
  union Out { uint32_t u[4]; b8 v; } out[3];
  __device__ __forceinline__ void first(int i, int part) {   // pair i: this part, and the remainders
    const f32x2 v = {x[2 * i], x[2 * i + 1]};
    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    out[part].u[i] = h;
    x[2 * i] -= __uint_as_float(h << 16);
    x[2 * i + 1] -= __uint_as_float(h & 0xFFFF0000u);
    pin(x[2 * i]);
    pin(x[2 * i + 1]);
    pin(out[part].u[i]);
  }
  __device__ __forceinline__ void rest(int i) {
    first(i, 1);
    const f32x2 v = {x[2 * i], x[2 * i + 1]};
    out[2].u[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    pin(out[2].u[i]);
  }
  __device__ __forceinline__ void step(int i) {
    if (i == 0) first(0, 0);
    if (i == 1) first(1, 0);
    if (i == 2) { rest(0); first(2, 0); }
    if (i == 3) rest(1);
    if (i == 4) first(3, 0);
    if (i == 5) { rest(2); rest(3); }
  }
  __device__ __forceinline__ Parts parts() const { return Parts{{out[0].v, out[1].v, out[2].v}}; }
};
// Six MFMAs of one 32 x 32 product, side(i) in the shadow of the i-th; nothing moves across their borders.
template <typename F>
__device__ __forceinline__ void mul32_slots(const Parts& a, const Parts& b, f32x16& c, F side) {
  constexpr int ia[6] = {0, 2, 1, 0, 1, 0}, ib[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
  for (int i = 0; i < 6; i++) {
    c = mfma(a.p[ia[i]], b.p[ib[i]], c);
    side(i);
    pin(c);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// lambda^e for e >= 0, with the logarithm to twice the working precision: l2 + l2lo = log2(lambda)
struct Decay {
  float l2, l2lo;
  __device__ __forceinline__ explicit Decay(float lambda) {
    const double d = log2((double)lambda);
    l2 = (float)d;
    l2lo = (float)(d - (double)l2);
  }
  __device__ __forceinline__ float pow(int e) const {
    const float x = (float)e, p = l2 * x;
    const float rest = fmaf(l2, x, -p) + l2lo * x;
    const float y = exp2f(p);
    return fmaf(y * 0.6931471805599453f, rest, y);
  }
};

template <int D>
__device__ __forceinline__ int state_index_f32(int dvt, int l32, int hh, int t, int v, bool transposed) {
  const int dk = 32 * t + 16 * (v >> 3) + 8 * hh + (v & 7);
  const int dv = 32 * dvt + l32;
  return transposed ? dv * D + dk : dk * D + dv;
}

template <int D, bool STATE_ONLY>
struct Lds {
  static constexpr int PROW = 40;   // elements per row of a score plane (80 bytes: 16 rows in 16 bank groups)
  __attribute__((aligned(1024))) __bf16 x[STATE_ONLY ? 1 : 3][STATE_ONLY ? 512 : kBF * D];
  __attribute__((aligned(1024))) __bf16 y[3][kBF * D];
  __attribute__((aligned(16))) __bf16 p[STATE_ONLY ? 1 : 3][STATE_ONLY ? 8 : kBF * PROW];   // [position r][c]
  __attribute__((aligned(16))) float wz[kBF];          // weight of a row of Z in the state update
  float red[STATE_ONLY ? 1 : kBF * (D / 32)];          // Norm epilogue: partial sums of squares, [row][wave]
  int good;                                            // blocks before a value that is not finite
};

struct Place {   // what a workgroup works on; the same for all its lanes
  int which, chain, chunk, bi, hi, n;
  int64_t base;
};

// One walk over the workgroup's chunk: the scan, or (STATE_ONLY) the chunk-state pre-pass (only Y, Z and the state update).
// D / 32 waves.  Leaves the state after the chunk, times 2^32 if not FP32, in kv.
// FP32 = false: on split operands; returns -1, or (to all waves) the number of blocks, in the order of the walk, whose
// outputs are in order when the chunk has to be walked again for the others and the state.  FP32 = true: on the fp32 matrix
// instructions; outputs of the blocks from number `from` on are stored.
template <int D, bool REV, bool STATE_ONLY, bool FP32>
__device__ __forceinline__ int walk(const ScanParams& p, Lds<D, STATE_ONLY>& lds, const Place& place, f32x16 (&kv)[D / 32],
                                    int from = 0) {
  constexpr int B = kBF;
  constexpr int NT = D / 32;          // waves; 32-wide feature tiles
  constexpr int KS = D / 16;          // k-steps along the features
  constexpr int CPR = D / 8;          // 8-feature pieces per row
  constexpr int TILE = B * D;         // elements per plane
  constexpr int PROW = Lds<D, STATE_ONLY>::PROW;
  constexpr float UP = FP32 ? 1.f : kUp;
  auto& sX = lds.x;
  auto& sY = lds.y;
  auto& sP = lds.p;
  auto& sWz = lds.wz;
  auto& sRed = lds.red;

  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // (nothing of one walk is kept in registers for the other)
  const int w = tid >> 6, l = tid & 63, l32 = l & 31, hh = l >> 5;
  const int dvt = w;
  const int which = place.which, chain = place.chain, chunk = place.chunk, bi = place.bi, hi = place.hi, n = place.n;
  const int64_t base = place.base;
  const uint32_t stride_n = (uint32_t)p.stride_n;

  const int nblocks = (n + B - 1) / B;
  const int cb = p.chunk_tokens / B;
  const int blk_lo = chunk * cb;
  const int blk_hi = min(blk_lo + cb, nblocks);
  const int nblk = max(blk_hi - blk_lo, 0);

  // Buffer descriptors over the chain's rows: rows past the end load as zeros and their stores are dropped.
  const uint32_t chain_bytes = n > 0 ? ((uint32_t)(n - 1) * stride_n + D) * 4u : 0u;
  auto rows_of = [&](const void* ptr) __attribute__((always_inline)) {
    return make_rsrc(reinterpret_cast<const float*>(ptr) + base, chain_bytes);
  };
  const __amdgpu_buffer_rsrc_t gx = rows_of(STATE_ONLY ? p.y[0] : which ? p.x[1] : p.x[0]);
  const __amdgpu_buffer_rsrc_t gy = rows_of(which ? p.y[1] : p.y[0]);
  const __amdgpu_buffer_rsrc_t gz = rows_of(which ? p.z[1] : p.z[0]);
  const __amdgpu_buffer_rsrc_t gw = rows_of(STATE_ONLY ? p.y[0] : which ? p.w[1] : p.w[0]);

  // ---- tile loads: this thread's two 8-feature pieces of X and Y (rows r0 and r0 + 16), this lane's column of Z
  const int r0 = tid / CPR, ch = tid % CPR;
  const int plane_at = r0 * D + 8 * (ch ^ swz<D>(r0));   // swz depends on row % 16: the second piece is 16 D further
  float px[2][8], py[2][8], pz[16];
  auto load8 = [&](const __amdgpu_buffer_rsrc_t& g, uint32_t off, float (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const i32x4 r = __builtin_amdgcn_raw_buffer_load_b128(g, off + 16u * i, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; j++) x[4 * i + j] = __int_as_float(r[j]);
    }
  };
  auto load_block = [&](int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const uint32_t off = ((uint32_t)(blk * B + r0 + 16 * i) * stride_n + 8u * ch) * 4u;
      load8(gy, off, py[i]);
      if (!STATE_ONLY) load8(gx, off, px[i]);
    }
    uint32_t zoff = ((uint32_t)(blk * B + 4 * hh) * stride_n + (uint32_t)(32 * dvt + l32)) * 4u;
    pin(zoff);   // the sixteen offsets are made here: kept across blocks they would be sixteen registers
#pragma unroll
    for (int v = 0; v < 16; v++)
      pz[v] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(gz, zoff + (uint32_t)(8 * (v >> 2) + (v & 3)) * stride_n * 4u, 0, 0));
  };
  float zr[16];   // the Z column of the block whose planes are in LDS
  auto write_planes = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 16; v++) zr[v] = pz[v];
#pragma unroll
    for (int i = 0; i < 2; i++) {
#pragma unroll
      for (int j = 0; j < 8; j++) {
        py[i][j] *= kUp;
        if (!STATE_ONLY) px[i][j] *= kUp;
      }
      const Parts y = split8(py[i]);
#pragma unroll
      for (int k = 0; k < 3; k++) *reinterpret_cast<b8*>(&sY[k][plane_at + 16 * D * i]) = y.p[k];
      if (!STATE_ONLY) {
        const Parts x = split8(px[i]);
#pragma unroll
        for (int k = 0; k < 3; k++) *reinterpret_cast<b8*>(&sX[k][plane_at + 16 * D * i]) = x.p[k];
      }
    }
  };

  // ---- running state slice S[:, dv tile]: NT accumulator tiles (key-feature tiles), fp32
  const Decay lam(p.lambda[hi]);
#pragma unroll
  for (int t = 0; t < NT; t++) kv[t] = zero16();
  if constexpr (!STATE_ONLY) {
    // kv <- decay kv + UP^2 * a d x d state (row = y feature, or transposed: eight consecutive elements of a stored row)
    auto add_state = [&](const float* gs, bool tr, float decay) __attribute__((always_inline)) {
      uint32_t at = (uint32_t)state_index_f32<D>(dvt, l32, hh, 0, 0, tr);
      pin(at);   // one lane offset, the rest is uniform: not sixteen addresses per tile
#pragma unroll
      for (int t = 0; t < NT; t++) {
        float x[16];
        if (tr) {
#pragma unroll
          for (int v = 0; v < 16; v += 4) {
            const f32x4 r = *reinterpret_cast<const f32x4*>(gs + (32 * t + 16 * (v >> 3) + (v & 7)) + at);
#pragma unroll
            for (int i = 0; i < 4; i++) x[v + i] = r[i];
          }
        } else {
#pragma unroll
          for (int v = 0; v < 16; v++) x[v] = (gs + (32 * t + 16 * (v >> 3) + (v & 7)) * D)[at];
        }
#pragma unroll
        for (int v = 0; v < 16; v++) kv[t][v] = fmaf(decay, kv[t][v], x[v] * (UP * UP));
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    const float* const init = which ? p.init[1] : p.init[0];
    const bool init_tr = (p.init_transposed >> which) & 1, state_tr = (p.state_transposed >> which) & 1;
    if (init != nullptr && (p.states == nullptr || p.self_prefix != 0)) add_state(init + (int64_t)chain * (D * D), init_tr, 0.f);
    if (p.states != nullptr && p.self_prefix == 0) {
      add_state(p.states + ((int64_t)chain * p.nchunks + chunk) * (D * D), state_tr, 0.f);
    } else if (p.states != nullptr) {   // the local states of the chunks this scan passes before (ScanParams::self_prefix)
      const int nch = min((nblocks + cb - 1) / cb, p.nchunks);   // (a longer sequence than planned for: the caller's error)
      const float lam_full = lam.pow(p.chunk_tokens), lam_last = lam.pow(n - (nch - 1) * p.chunk_tokens);
#pragma unroll 1
      for (int i = 0; i < (REV ? nch - 1 - chunk : chunk); i++) {
        const int j = REV ? nch - 1 - i : i;
        add_state(p.states + ((int64_t)chain * p.nchunks + j) * (D * D), state_tr, j == nch - 1 ? lam_last : lam_full);
      }
    }
  }

  // ---- decay weights: of the rows of Z in the state update (LDS), of the carried state at this lane's position, of the
  // quarters of the score tile S^T[c][r] that this wave computes (lane: position
  // r = 16 rq + l % 16, elements i: c = 16 cq + 4 (l / 16) + i).
  if (tid < B) sWz[tid] = UP * lam.pow(REV ? tid + 1 : B - 1 - tid);
  if (!FP32 && tid == 0) lds.good = nblk + 1;
  const float lamB = uniform(lam.pow(B));
  const float inter_scale = lam.pow(REV ? B - 1 - l32 : l32 + 1);
  constexpr int NQ = 4 / NT;   // quarters per wave: w, w + NT
  const int l16 = l & 15, g4 = l >> 4;
  float dg[STATE_ONLY ? 1 : NQ][4];
  if (!STATE_ONLY && !FP32) {
#pragma unroll
    for (int u = 0; u < NQ; u++) {
      const int q = w + NT * u, cq = q & 1, rq = q >> 1;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int c = 16 * cq + 4 * g4 + i, r = 16 * rq + l16, e = REV ? c - r : r - c;
        dg[u][i] = e >= 0 ? lam.pow(e) : 0.f;
      }
    }
    for (int i = tid; i < 3 * B * PROW / 2; i += 2 * D) reinterpret_cast<uint32_t*>(&sP[0][0])[i] = 0u;   // the empty quarter stays zero
  }

  if (!FP32 && nblk > 0) load_block(REV ? blk_hi - 1 : blk_lo);

  // ---- LDS addresses: row fragments (32 rows x 16 features; 16 rows x 32 features), transposing reads
  const int rowk = l32 * D + 8 * (hh ^ swz<D>(l32));       // 32-row fragment of k-step ks: rowk ^ 16 ks
  const int rowq = l16 * D + 8 * (g4 ^ swz<D>(l16));       // 16-row fragment of k-step ks: rowq ^ 32 ks (+ 16 D rows)
  int tr0, tr1;
  {
    const int g2 = (l >> 4) & 1, piece = l & 3;
    const int trc = 2 * g2 + (piece & 1), trh = 4 * (piece >> 1);   // bits 2 and 3 of the column exchanged
    const int ra = 4 * hh + (l16 >> 2), rb = ra + 8;
    tr0 = ra * D + 8 * (trc ^ swz<D>(ra)) + trh;
    tr1 = rb * D + 8 * (trc ^ swz<D>(rb)) + trh;
  }
  auto read_parts = [&](const __bf16 (*plane)[TILE], int at) __attribute__((always_inline)) {
    Parts r;
#pragma unroll
    for (int k = 0; k < 3; k++) r.p[k] = *reinterpret_cast<const b8*>(&plane[k][at]);
    return r;
  };
  auto read_ycols = [&](int q, int t) __attribute__((always_inline)) {   // rows 16 q .. + 15, key-feature tile t
    Parts r;
#pragma unroll
    for (int k = 0; k < 3; k++) {
      union { struct { s16x4 lo, hi; } s; b8 v; } u;
      u.s.lo = lds_read_tr(&sY[k][16 * q * D + (tr0 ^ (32 * t))]);
      u.s.hi = lds_read_tr(&sY[k][16 * q * D + (tr1 ^ (32 * t))]);
      r.p[k] = u.v;
    }
    return r;
  };

  auto block_at = [&](int it) { return REV ? blk_hi - 1 - it : blk_lo + it; };

  // Output of a block: lane = position l32, elements v = 4 g .. 4 g + 3 are value features 32 dvt + 8 g + 4 hh .. + 3.
  // One workgroup barrier, before which the caller is done with the block's LDS.
  auto emit = [&](f32x16& w, int blk, bool keep) __attribute__((always_inline)) {
    const int pos = keep ? blk * B + l32 : n;
    // Rows of 16 lanes exchange pieces so that an instruction stores whole 64-byte pieces of sixteen positions, which a
    // streaming store needs (16 bytes a lane in 32 rows: 1.25 times the time of the whole launch).  Batch 4, H 16, n 2048,
    // d 128, forward + backward, against 16-byte pieces through the caches: 433 -> 425 us replayed from a graph; as a program's
    // calls, the two in turn on three boxes, 0.5 to 0.9 %.
    auto store_rows = [&]() __attribute__((always_inline)) {
      const uint32_t row = (uint32_t)((keep ? blk * B : n) + (l32 & 15));
      const uint32_t off = (row * stride_n + (uint32_t)(32 * dvt + 8 * (l32 >> 4) + 4 * hh)) * 4u;
#pragma unroll
      for (int u = 0; u < 2; u++) {   // pieces 2 u and 2 u + 1: lanes 16 .. 31 of the first <-> lanes 0 .. 15 of the second
        u32x4 o[2];
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const u32x2 x = __builtin_amdgcn_permlane16_swap(__float_as_uint(w[8 * u + i]), __float_as_uint(w[8 * u + 4 + i]), false, false);
          o[0][i] = x[0];
          o[1][i] = x[1];
        }
#pragma unroll
        for (int i = 0; i < 2; i++)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, o[i]), gw, off + 64u * u + 64u * i * stride_n, 0, 18);
      }
    };
    if (p.rstd != nullptr) {   // Norm epilogue (eq. (2)); the sums meet under the barrier
      norm_publish<NT>(w, sRed, l32, hh, dvt);
      lds_barrier();
      const float r = norm_collect<NT>(sRed, l32, 1.f / (float)D, p.eps);
#pragma unroll
      for (int v = 0; v < 16; v++) w[v] *= r;
      if (dvt == 0 && hh == 0 && pos < n) p.rstd[rstd_chain_offset(p, bi, hi) + pos] = r;
      store_rows();
    } else {
      store_rows();
      lds_barrier();
    }
  };

  if constexpr (!FP32) {
    if (nblk > 0) write_planes();
    lds_barrier();

    float worst = 0.f;   // largest magnitude among this lane's outputs so far; NaN if one is NaN
    int good = 0;        // blocks up to which that is finite

    for (int it = 0; it < nblk; it++) {
      const int blk = block_at(it);
      const bool has_next = it + 1 < nblk;
      if (has_next) load_block(REV ? blk - 1 : blk + 1);

      // The body is a sequence of slots: the MFMAs of one product, in their shadow the LDS reads and the splits of the
      // next one (left alone the compiler puts every split in front of the product that takes it).
      f32x16 acc = zero16();
      Parts yt[2], zd, zf[2];
      // Pre-pass: only the state after the last block is wanted, so every block's contribution carries its whole decay up
      // front.
      const float up = STATE_ONLY ? uniform(lam.pow(B * (nblk - 1 - it))) : 1.f;
      Splitter sp;
      auto z_into = [&](int q, bool decayed) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const f32x4 wt = *reinterpret_cast<const f32x4*>(&sWz[16 * q + 8 * h + 4 * hh]);
#pragma unroll
          for (int j = 0; j < 4; j++)
            sp.x[4 * h + j] = zr[8 * q + 4 * h + j] * (!decayed ? kUp : STATE_ONLY ? wt[j] * up : wt[j]);
        }
      };
      if constexpr (!STATE_ONLY) {
        auto state_into = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
          for (int j = 0; j < 8; j++) sp.x[j] = kv[ks >> 1][8 * (ks & 1) + j];
        };
        // score quarters S^T[c][r] = sum_k Y[c][k] X[r][k]  (the empty quarter: computed by the wave that would idle, not used)
        f32x4 s[NQ];
        Parts xa[2] = {read_parts(sX, rowk), {}};
#pragma unroll
        for (int u = 0; u < NQ; u++) {
          const int q = w + NT * u, cq = q & 1, rq = q >> 1;
          s[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < D / 32; ks++)
            s[u] = mul16(read_parts(sY, 16 * cq * D + (rowq ^ (32 * ks))), read_parts(sX, 16 * rq * D + (rowq ^ (32 * ks))), s[u]);
        }
        state_into(0);
#pragma unroll
        for (int i = 0; i < 6; i++) sp.step(i);
        Parts sa = sp.parts();
#pragma unroll
        for (int u = 0; u < NQ; u++) pin(s[u]);
        __builtin_amdgcn_sched_barrier(0);
        // inter-block part W^T[dv][r] = sum_dk State[dk][dv] X[r][dk], state straight from its registers
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
          mul32_slots(sa, xa[ks & 1], acc, [&](int i) __attribute__((always_inline)) {
            if (i == 0) {
              if (ks + 1 < KS) {
                xa[(ks + 1) & 1] = read_parts(sX, rowk ^ (16 * (ks + 1)));
                state_into(ks + 1);
              } else {
                yt[0] = read_ycols(0, 0);
                z_into(0, true);
              }
            }
            sp.step(i);
            if ((ks & 1) && i < 4) {   // both operands of state tile ks / 2 are made
#pragma unroll
              for (int v = 0; v < 4; v++) {
                float y = kv[ks >> 1][4 * i + v] * lamB;
                pin(y);
                kv[ks >> 1][4 * i + v] = y;
              }
            }
          });
          if (ks < NQ) {   // the quarter's mask and decay, to LDS: row r, columns in the order of the intra-block operand
            const int q = w + NT * ks, cq = q & 1, rq = q >> 1;
            if (REV ? cq >= rq : cq <= rq) {
              uint32_t part[3][2];
#pragma unroll
              for (int i = 0; i < 2; i++)
                split2(s[ks][2 * i] * dg[ks][2 * i], s[ks][2 * i + 1] * dg[ks][2 * i + 1], part[0][i], part[1][i], part[2][i]);
              const int at = (16 * rq + l16) * PROW + 16 * cq + 8 * (g4 & 1) + 4 * (g4 >> 1);
#pragma unroll
              for (int k = 0; k < 3; k++) *reinterpret_cast<u32x2*>(&sP[k][at]) = u32x2{part[k][0], part[k][1]};
            }
          }
          sa = sp.parts();
        }
      } else {
        yt[0] = read_ycols(0, 0);
        z_into(0, true);
#pragma unroll
        for (int i = 0; i < 6; i++) sp.step(i);
      }
      zd = sp.parts();
      // state slice <- lambda^B state + Y^T decay(Z)
#pragma unroll
      for (int u = 0; u < 2 * NT; u++) {
        const int t = u % NT;
        mul32_slots(yt[u & 1], zd, kv[t], [&](int i) __attribute__((always_inline)) {
          if (i == 0 && u + 1 < 2 * NT) yt[(u + 1) & 1] = read_ycols((u + 1) / NT, (u + 1) % NT);
          if (u == NT - 1) {
            if (i == 0) z_into(1, true);
            sp.step(i);
          }
          if constexpr (!STATE_ONLY) {
            if (u == 0 && i < 4) {   // the carried part takes the decay at this lane's position
#pragma unroll
              for (int v = 0; v < 4; v++) {
                float y = acc[4 * i + v] * inter_scale;
                pin(y);
                acc[4 * i + v] = y;
              }
            }
            if (u >= NT && u < NT + 2) {   // Z as it is, for the intra-block product
              if (i == 0) z_into(u - NT, false);
              sp.step(i);
            }
          }
        });
        if (u == NT - 1) zd = sp.parts();
        if (!STATE_ONLY && u >= NT && u < NT + 2) zf[u - NT] = sp.parts();
      }
      lds_barrier();   // every wave has read this block's planes, the score tile is complete
      if (has_next) write_planes();
      if constexpr (!STATE_ONLY) {
        // intra-block part Z^T P^T
#pragma unroll
        for (int q = 0; q < 2; q++) {
          Parts pd;
#pragma unroll
          for (int k = 0; k < 3; k++) pd.p[k] = *reinterpret_cast<const b8*>(&sP[k][l32 * PROW + 16 * q + 8 * hh]);
          acc = mul32(zf[q], pd, acc);
        }
#pragma unroll
        for (int v = 0; v < 16; v++) {
          worst = __builtin_elementwise_maximum(worst, __builtin_fabsf(acc[v]));
          acc[v] *= 1.f / (kUp * kUp * kUp);
        }
        good += worst < __builtin_inff() ? 1 : 0;
        emit(acc, blk, true);
      } else {
        lds_barrier();
      }
    }

    // Everything that left the range of the scaled parts, Inf and NaN among the inputs included, has made an output or an
    // element of the state infinite or NaN by now.  Such a chunk is walked again from its start, in fp32 throughout.
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int v = 0; v < 16; v++) worst = __builtin_elementwise_maximum(worst, __builtin_fabsf(kv[t][v]));
    if (!(worst < __builtin_inff())) atomicMin(&lds.good, good);
    lds_barrier();
    const int first = __builtin_amdgcn_readfirstlane(lds.good);
    if (first <= nblk) return first;
  } else {
    float* const fY = reinterpret_cast<float*>(&sY[0][0]);
    float* const fX = STATE_ONLY ? fY : reinterpret_cast<float*>(&sX[0][0]);
    static_assert(sizeof(lds.y) >= sizeof(float) * TILE && (STATE_ONLY || sizeof(lds.x) >= sizeof(float) * TILE),
                  "fp32 tiles in the planes' place");
    // feature f of tile row r: 16-byte pieces swizzled by r % 16
    auto at = [](int r, int f) { return r * D + ((((f >> 2) ^ (r & 15)) << 2) | (f & 3)); };
    lds_barrier();   // the weights are written
#pragma unroll 1
    for (int it = 0; it < nblk; it++) {
      const int blk = block_at(it);
      // made from the lane number in every block: kept over the loop the addresses and weights would not fit the registers
      int lo = l;
      asm volatile("" : "+v"(lo));
      const int row = lo & 31, half = lo >> 5;
      const int col = (row & 19) | ((row & 4) << 1) | ((row & 8) >> 1);   // feature of state row `row`: bits 2 and 3 exchanged
      load_block(blk);   // (the block before ended with a barrier: its tiles are free)
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 8; j += 4) {
          *reinterpret_cast<f32x4*>(&fY[at(r0 + 16 * i, 8 * ch + j)]) = f32x4{py[i][j], py[i][j + 1], py[i][j + 2], py[i][j + 3]};
          if (!STATE_ONLY)
            *reinterpret_cast<f32x4*>(&fX[at(r0 + 16 * i, 8 * ch + j)]) = f32x4{px[i][j], px[i][j + 1], px[i][j + 2], px[i][j + 3]};
        }
      lds_barrier();
      f32x16 acc = zero16();
      if constexpr (!STATE_ONLY) {
        f32x16 st = zero16();
#pragma unroll
        for (int t = 0; t < NT; t++)   // inter-block part, two key features per instruction: state register v's
#pragma unroll
          for (int v = 0; v < 16; v += 4) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(&fX[at(row, 32 * t + 16 * (v >> 3) + 8 * half + (v & 7))]);
#pragma unroll
            for (int i = 0; i < 4; i++) acc = mfma_f32(kv[t][v + i], x[i], acc);
            __builtin_amdgcn_sched_barrier(0);   // (few operands in flight: there are no registers for more)
          }
#pragma unroll
        for (int j = 0; j < D / 8; j++) {   // scores S^T[c][r]
          const f32x4 x = *reinterpret_cast<const f32x4*>(&fX[at(row, 8 * j + 4 * half)]);
          const f32x4 y = *reinterpret_cast<const f32x4*>(&fY[at(row, 8 * j + 4 * half)]);
#pragma unroll
          for (int i = 0; i < 4; i++) st = mfma_f32(y[i], x[i], st);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int v = 0; v < 16; v++) acc[v] *= inter_scale;
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int c = 8 * (v >> 2) + 4 * half + (v & 3), e = REV ? c - row : row - c;
          acc = mfma_f32(pz[v], st[v] * (e >= 0 ? lam.pow(e) : 0.f), acc);
        }
      }
#pragma unroll
      for (int t = 0; t < NT; t++)
#pragma unroll
        for (int v = 0; v < 16; v++) kv[t][v] *= lamB;
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const int c = 8 * (v >> 2) + 4 * half + (v & 3);
        const float zw = pz[v] * sWz[c];
#pragma unroll
        for (int t = 0; t < NT; t++) kv[t] = mfma_f32(fY[at(c, 32 * t + col)], zw, kv[t]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (STATE_ONLY) lds_barrier();
      else emit(acc, blk, it >= from);
    }
  }

  return -1;
}

// Scan kernel (STATE_ONLY = false) and chunk-state pre-pass (STATE_ONLY = true: the local state of the chunk is written to
// p.states).  D / 32 waves.  (The parameters by value: the compiler then loads them together at the kernel's start.  Through a reference
// kept by a lambda they were loaded one after another where they are used, 0.5 to 1 us a launch more: 8 chains of 154, head_dim 128,
// forward 25.7 -> 26.3 us; through a plain reference the kernels of head_dim 64 spill scalar registers.)
template <int D, bool REV, bool STATE_ONLY>
__device__ __forceinline__ void scan_f32(const ScanParams p, int wg, const unsigned grid, Lds<D, STATE_ONLY>& lds) {
  constexpr int NT = D / 32;
  Place at;
  at.which = 0;
  if (!STATE_ONLY && p.nscan == 2) {   // two scans that read the same tiles: eight workgroups apart, on one XCD
    if (((grid >> 1) & 7) == 0) {
      at.which = (wg >> 3) & 1;
      wg = ((wg >> 4) << 3) | (wg & 7);
    } else {
      at.which = wg & 1;
      wg >>= 1;
    }
  }
  at.chain = wg / p.nchunks;
  at.chunk = wg % p.nchunks;
  at.bi = at.chain / p.heads;
  at.hi = at.chain % p.heads;
  chain_extent(p, at.bi, at.hi, at.base, at.n);
  const int first = at.chunk * p.chunk_tokens;
  if (!STATE_ONLY && first >= at.n) return;
  // pre-pass: the chunk a scan of THIS chain passes last has no successor (packed batch: chains of different lengths)
  if (STATE_ONLY && (REV ? (at.chunk == 0) : (first + p.chunk_tokens >= at.n))) return;

  f32x16 kv[NT];
  float down = 1.f / (kUp * kUp);
  const int from = walk<D, REV, STATE_ONLY, false>(p, lds, at, kv);
  if (from >= 0) {
    walk<D, REV, STATE_ONLY, true>(p, lds, at, kv, from);
    down = 1.f;
  }

  // the chunk's local state (pre-pass) or the state after the chain's last block (on request)
  float* gf = nullptr;
  bool trf = false;
  if (STATE_ONLY) {
    gf = p.states + ((int64_t)at.chain * p.nchunks + at.chunk) * (D * D);
  } else if ((at.which ? p.fin[1] : p.fin[0]) != nullptr && (REV ? at.chunk == 0 : at.chunk == p.nchunks - 1)) {
    gf = (at.which ? p.fin[1] : p.fin[0]) + (int64_t)at.chain * (D * D);
    trf = (p.fin_transposed >> at.which) & 1;
  }
  if (gf != nullptr) {
    const int l = (int)threadIdx.x & 63, dvt = (int)threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int v = 0; v < 16; v++) gf[state_index_f32<D>(dvt, l & 31, l >> 5, t, v, trf)] = kv[t][v] * down;
  }
}

template <int D, bool REV, bool STATE_ONLY>
__global__ __launch_bounds__(2 * D) __attribute__((amdgpu_waves_per_eu(2, 2))) void scan_f32_kernel(ScanParams p) {
  __shared__ Lds<D, STATE_ONLY> lds;
  scan_f32<D, REV, STATE_ONLY>(p, (int)blockIdx.x, gridDim.x, lds);
}

// Both families of a backward pass's chunk states in one launch: the first half of the workgroups the forward ones, the second half
// the reverse ones.  Each alone has at most one workgroup of four waves per compute unit at head_dim 128, bound by its issue, which a
// second one fills.  Forward + backward with one launch against two, the states the same bits: d 128, 48 chains of 1500 287 -> 274 us,
// 64 of 1024, 2048 246 -> 234, 431 -> 415, 128 of 1024 418 -> 388; d 64, 4 chains of 1000 78 -> 71, 64 of 2048 211 -> 206, 96 even.
template <int D>
__global__ __launch_bounds__(2 * D) __attribute__((amdgpu_waves_per_eu(2, 2))) void chunk_state_pair_f32_kernel(ScanParams fwd, ScanParams rev) {
  __shared__ Lds<D, true> lds;
  const int units = (int)gridDim.x / 2, wg = (int)blockIdx.x;
  if (wg < units) scan_f32<D, false, true>(fwd, wg, (unsigned)units, lds);
  else            scan_f32<D, true, true>(rev, wg - units, (unsigned)units, lds);
}

template <bool STATE_ONLY>
hipError_t launch(int head_dim, bool reverse, const ScanParams& p, hipStream_t s) {
  const int64_t grid = (int64_t)p.batch * p.heads * p.nchunks * (STATE_ONLY ? 1 : p.nscan);
  if (grid == 0 || p.n == 0) return hipSuccess;
  const dim3 g((unsigned)grid), b(2 * head_dim);
  if (head_dim == 128) {
    if (reverse) hipLaunchKernelGGL((scan_f32_kernel<128, true, STATE_ONLY>), g, b, 0, s, p);
    else         hipLaunchKernelGGL((scan_f32_kernel<128, false, STATE_ONLY>), g, b, 0, s, p);
  } else {
    if (reverse) hipLaunchKernelGGL((scan_f32_kernel<64, true, STATE_ONLY>), g, b, 0, s, p);
    else         hipLaunchKernelGGL((scan_f32_kernel<64, false, STATE_ONLY>), g, b, 0, s, p);
  }
  return hipGetLastError();
}

}  // namespace

int block_size_f32(int) { return kBF; }

hipError_t launch_scan_f32(int head_dim, bool reverse, const ScanParams& p, hipStream_t s) {
  return launch<false>(head_dim, reverse, p, s);
}

hipError_t launch_chunk_state_pair_f32(int head_dim, const ScanParams& fwd, const ScanParams& rev, hipStream_t s) {
  const int64_t grid = 2 * (int64_t)fwd.batch * fwd.heads * fwd.nchunks;
  if (grid == 0 || fwd.n == 0) return hipSuccess;
  if (grid * 2 * head_dim > 0xFFFFFFFFll) return hipErrorInvalidValue;   // work-items (la2_api.hip sends no such call here)
  const dim3 g((unsigned)grid), b(2 * head_dim);
  if (head_dim == 128) hipLaunchKernelGGL((chunk_state_pair_f32_kernel<128>), g, b, 0, s, fwd, rev);
  else                 hipLaunchKernelGGL((chunk_state_pair_f32_kernel<64>), g, b, 0, s, fwd, rev);
  return hipGetLastError();
}

hipError_t launch_chunk_states_f32(int head_dim, bool reverse, const ScanParams& p, hipStream_t s) {
  return launch<true>(head_dim, reverse, p, s);
}

}  // namespace la2

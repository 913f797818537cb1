// Short sequences on few chains, 16-bit data, head_dim 64 / 128, gfx950: every output row block looks at all the positions it
// depends on itself, so that a forward or a backward pass is ONE launch.
//
// The block recurrence walks a chain block by block, and a chain that is cut into chunks needs the states at their starts from
// launches before: on a few chains of a few hundred positions that is a handful of dependent launches of 8 to 20 us each, on a
// device that is mostly idle.  Here a workgroup owns 64 positions of one chain and forms their rows as masked products
//     W = [(X Y^T) * M] Z        (M: decay lambda^|t - s| on one side of the diagonal, 0 on the other)
// over all the positions on that side: more arithmetic in all (it grows with the square of the length), but no position waits
// for another workgroup.  Beside the scans of a pass (forward: one; backward: dQ, and dV, dK with the transposed mask) the
// same launch has workgroups for the states that are handed out.
//
// Work split: four waves, two row tiles of 32 x two key groups; a step is 64 positions of Y and Z, a tile of 32 per key
// group, loaded straight into LDS (two buffers: the next step's tiles are on their way while one is used; one barrier a step).
// The key groups' sums meet in LDS at the end, in the tiles' place, where the row is complete for the Norm epilogue.  Scores,
// mask and operands as in the scan kernels: 16-bit operands, fp32 sums, the masked scores rounded to 16 bits once; what is
// rounded carries the decay of one tile at most where the type's range asks for that (fp16 scores, all states).
// MFMA and LDS layouts: la2_bf16_common.h.
//
// What bounds it: a workgroup's own instruction stream.  A step takes a lone workgroup about 0.65 us (d 128; 0.4 at d 64), of
// which the products are 0.22 (16 per wave) and the issue of its eight direct loads as much again; start, first loads, the sums
// and the stores are about 4 us.  64 KiB (32 at d 64) of LDS, so two (four) workgroups share a compute unit and fill each
// other's gaps.  Tried: eight waves with four key groups, one workgroup per unit at d 128 (a lone long chain 20 % faster, full
// launches 20-40 % slower), two waves (the reverse: 10 % either way), three and four buffers (no change: not the loads'
// latency), all LDS reads ahead of the products (no change), the loads between the products (8 % slower: they come later),
// the non-temporal hint on the loads (15 % slower: other workgroups read the same tiles).
// Forward / backward of 16 chains, against the block recurrence (chunk-state pre-pass and scans), us from a replayed graph, bf16:
// d 128, n 128: 8.1 -> 6.4, 18.5 -> 6.7; n 512: 20.0 -> 10.7, 48.3 -> 13.0; n 1024: 23.1 -> 16.8, 48.9 -> 25.9;
// d 64, n 128: 6.5 -> 5.1, 12.9 -> 5.2; n 512: 14.5 -> 7.7, 30.0 -> 8.5; n 1024: 14.7 -> 11.3, 27.4 -> 13.7.
// fp16 takes 8 to 15 % longer, d 64 up to 25 (the scores' scales, below).  With the state handed out, 16 chains of 777 positions,
// d 128: 23.8 -> 14.8 (18.4 with one workgroup per chain's state).  A start state is read by every row block: 3 us more at d 128.
#include "la2_bf16_common.h"

namespace la2 {
namespace {
using namespace bf16k;

constexpr int kRows = 64;              // output positions per workgroup
constexpr int kGroups = 2;             // key groups (a tile of 32 positions each)
constexpr int kStep = 32 * kGroups;    // positions of Y and Z per step
constexpr int kWaves = 2 * kGroups;    // two row tiles of 32 times the key groups

template <typename E, int D, bool NORM>
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 4 : 2) void short_scan_kernel(ShortParams p) {
  using C = Cfg<D, kStep>;
  constexpr int KS = C::KS, NT = C::NT, TILE = C::TILE;
  constexpr int DPW = C::DMA_PER_TILE / kWaves;   // direct loads per wave and tile
  constexpr bool F16 = std::is_same<E, _Float16>::value;
  __shared__ __attribute__((aligned(1024))) E sT[2][2][TILE];   // [buffer][Y, Z]
  static_assert(sizeof(sT) >= sizeof(float) * kGroups * kRows * D, "the key groups' sums take the tiles' place");
  float* const part = reinterpret_cast<float*>(&sT[0][0][0]);

  const int tid = threadIdx.x, l = tid & 63, l32 = l & 31, hh = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // Which chain and what of it.  Chains are the fast index (a chain's workgroups share an XCD's L2 where their number is a
  // multiple of eight); the long row blocks come first, before them the chains' states.
  const int chains = p.batch * p.heads;
  const int chain = (int)blockIdx.x % chains;
  int item = (int)blockIdx.x / chains;
  const int bi = chain / p.heads, hi = chain % p.heads;
  int n;
  int64_t base;
  if (p.cu_seqlens != nullptr) {
    const int first = p.cu_seqlens[bi];
    n = p.cu_seqlens[bi + 1] - first;
    base = (int64_t)first * p.stride_n + (int64_t)hi * p.stride_h;
  } else {
    n = p.n;
    base = (int64_t)bi * p.stride_b + (int64_t)hi * p.stride_h;
  }
  n = __builtin_amdgcn_readfirstlane(n);
  const uint32_t base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base);
  const uint32_t base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)base >> 32));
  base = (int64_t)(((uint64_t)base_hi << 32) | base_lo);
  constexpr int SWG = NT * NT / kWaves;   // workgroups for a chain's state: a 32 x 32 tile per wave
  const int state_part = p.fin != nullptr ? item : SWG;
  const bool is_state = state_part < SWG;
  if (p.fin != nullptr) item -= SWG;
  const int which = is_state ? 0 : item % p.nscan;
  const int rank = is_state ? 0 : item / p.nscan;
  const bool rev = is_state ? p.state_rev != 0 : ((p.rev >> which) & 1) != 0;
  const int nrb = (p.n + kRows - 1) / kRows;
  const int row0 = kRows * (rev ? rank : nrb - 1 - rank);
  if (!is_state && row0 >= n) return;
  const float l2 = log2f(p.lambda[hi]);
  const uint32_t stride_n = (uint32_t)p.stride_n;

  const void* const vy = is_state ? p.state_y : which == 0 ? p.y[0] : which == 1 ? p.y[1] : p.y[2];
  const void* const vz = is_state ? p.state_z : which == 0 ? p.z[0] : which == 1 ? p.z[1] : p.z[2];
  const char* const gy = reinterpret_cast<const char*>(reinterpret_cast<const E*>(vy) + base);
  const char* const gz = reinterpret_cast<const char*>(reinterpret_cast<const E*>(vz) + base);

  // The 32-position tiles it looks at, first_tile .. first_tile + ntiles - 1 (ntiles 0: an empty sequence's state)
  const int last_tile = n > 0 ? (n - 1) >> 5 : -1;
  const int first_tile = is_state || !rev ? 0 : row0 >> 5;
  const int end_tile = is_state || rev ? last_tile : min((row0 + kRows - 1) >> 5, last_tile);
  const int ntiles = end_tile - first_tile + 1;
  const int nsteps = (ntiles + kGroups - 1) / kGroups;
  // Steps run from the far end towards the rows (a state: towards the end that it is the state at)
  auto step_first = [&](int s) __attribute__((always_inline)) { return 32 * first_tile + kStep * (rev ? nsteps - 1 - s : s); };

  // Direct loads: wave w issues loads DPW w .. of a tile; lane l of load j fills 16-byte piece q = 64 j + l, row q / CPR,
  // which holds the row's piece (q % CPR) ^ swz(row).  Rows past the end: the last row's, zeroed after they have landed.
  int lrow[DPW];
  uint32_t lcol[DPW];
  const uint32_t wave_lds = 1024u * DPW * (uint32_t)w;
#pragma unroll
  for (int i = 0; i < DPW; i++) {
    const int q = 64 * (DPW * w + i) + l;
    lrow[i] = q / C::CPR;
    lcol[i] = 8u * (uint32_t)((q % C::CPR) ^ swz<D>(q / C::CPR));
  }
  auto issue = [&](int s) __attribute__((always_inline)) {
    const int first = step_first(s);
    E (*const buf)[TILE] = sT[s & 1];
#pragma unroll
    for (int i = 0; i < DPW; i++) {
      const uint32_t off = ((uint32_t)min(first + lrow[i], n - 1) * stride_n + lcol[i]) * 2u;
      dma16_shared(gy, off, (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_offset(&buf[0][0]) + wave_lds + 1024u * i)));
      dma16_shared(gz, off, (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_offset(&buf[1][0]) + wave_lds + 1024u * i)));
    }
  };
  // step s's tiles are there for all waves (and everybody is done with the step before)
  auto arrive = [&](int s) __attribute__((always_inline)) {
    const int first = step_first(s);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    if (first + kStep > n) {
#pragma unroll
      for (int i = 0; i < DPW; i++) {
        if (first + lrow[i] >= n) {
          const i32x4 z = {0, 0, 0, 0};
          char* const at = reinterpret_cast<char*>(&sT[s & 1][0][0]) + wave_lds + 1024u * i + 16u * l;
          *reinterpret_cast<i32x4*>(at) = z;
          *reinterpret_cast<i32x4*>(at + sizeof(E) * TILE) = z;
        }
      }
    }
    lds_barrier();
  };
  if (nsteps > 0) issue(0);
  const LaneAddr<D> la(l);

  if (is_state) {
    // State right behind the chain's last position (rev: entering its first): sum_c weight(c) y_c^T z_c + lambda^n init,
    // weight lambda^(n - 1 - c) (rev: lambda^(c + 1)).  As in the scans, z carries the decay inside its tile of 32 positions when
    // it is rounded to 16 bits and the sums carry the rest in fp32: in fp16 the whole decay would make it subnormal, or zero.
    const int dvt = (kWaves * state_part + w) / NT, dkt = w % NT;
    f32x16 acc = zero16();
    // element j's factor and, for rows 16 k .. 16 k + 15 of a tile, a lane's, no exponent negative; row of element j: 16 k + 4 hh +
    // 8 (j / 4) + j % 4
    float gj[8], gk[2];
#pragma unroll
    for (int j = 0; j < 8; j++) gj[j] = uniform(exp2f(l2 * (float)(rev ? 8 * (j >> 2) + (j & 3) : 11 - 8 * (j >> 2) - (j & 3))));
#pragma unroll
    for (int k = 0; k < 2; k++) gk[k] = exp2f(l2 * (float)(rev ? 16 * k + 4 * hh + 1 : 16 * (1 - k) + 4 * (1 - hh)));
    const float lam32 = uniform(exp2f(l2 * 32.f));
    for (int s = 0; s < nsteps; s++) {
      arrive(s);
      if (s + 1 < nsteps) issue(s + 1);
      const E* const tY = sT[s & 1][0];
      const E* const tZ = sT[s & 1][1];
#pragma unroll
      for (int g = 0; g < kGroups; g++) {
        const int tile = rev ? kGroups - 1 - g : g;
        const int valid = min(max(n - step_first(s) - 32 * tile, 0), 32);   // rows; those past them are zero
        const bool whole = rev || valid == 32;
        const float carry = whole ? lam32 : uniform(exp2f(l2 * (float)valid));
#pragma unroll
        for (int v = 0; v < 16; v++) acc[v] *= carry;
#pragma unroll
        for (int k = 0; k < 2; k++) {
          const int c0 = 32 * tile + 16 * k;
          const ex8<E> z = la.read_cols(tZ, c0, dvt);
          ex8<E> zd;
          if (whole) {
#pragma unroll
            for (int j = 0; j < 8; j++) zd[j] = (E)((float)z[j] * (gk[k] * gj[j]));
          } else {
#pragma unroll
            for (int j = 0; j < 8; j++)
              zd[j] = (E)((float)z[j] * fast_exp2(l2 * (float)max(valid - 1 - 16 * k - 4 * hh - 8 * (j >> 2) - (j & 3), 0)));
          }
          acc = mfma(la.read_cols(tY, c0, dkt), zd, acc);
        }
      }
    }
    const float lam_n = exp2f(l2 * (float)n);
    const float* const gi = p.state_init != nullptr ? p.state_init + (int64_t)chain * (D * D) : nullptr;
    float* const gf = p.fin + (int64_t)chain * (D * D);
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int at = state_index<D>(dvt, l32, hh, dkt, v, false);
      gf[at] = gi != nullptr ? fmaf(lam_n, gi[at], acc[v]) : acc[v];
    }
    return;
  }

  // ---- 64 output rows
  const int rh = w & 1, kg = w >> 1;
  const int r = row0 + 32 * rh + l32;   // this lane's position
  ex8<E> xf[KS];                        // its row of X (natural k-order), straight from global memory
  {
    const void* const vx = which == 0 ? p.x[0] : which == 1 ? p.x[1] : p.x[2];
    const E* const gx = reinterpret_cast<const E*>(vx) + base + (int64_t)min(r, n - 1) * stride_n + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) xf[ks] = *reinterpret_cast<const ex8<E>*>(gx + 16 * ks);
    if (r >= n) {
#pragma unroll
      for (int ks = 0; ks < KS; ks++) xf[ks] = ex8<E>{};
    }
  }
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) acc[t] = zero16();
  // the caller's start state: lambda^(r + 1) x_r S (rev: lambda^(n - 1 - r)), half of the key features per key group
  const float* init = which == 0 ? p.init[0] : which == 1 ? p.init[1] : p.init[2];
  if (init != nullptr) {
    init += (int64_t)chain * (D * D);
    const bool tr = (p.init_transposed >> which) & 1;
    const uint32_t lane = tr ? (uint32_t)(l32 * D + 8 * hh) : (uint32_t)(8 * hh * D + l32);   // (32-bit: no address pairs to spill)
#pragma unroll
    for (int kk = 0; kk < KS; kk++) {
      if (kk / (KS / kGroups) != kg) continue;   // (unrolled with a uniform condition: xf[] is indexed by constants)
#pragma unroll
      for (int t = 0; t < NT; t++) {
        ex8<E> a;
        if (tr) {
          const uint32_t at = lane + (uint32_t)(32 * t * D + 16 * kk);
          const f32x4 lo = *reinterpret_cast<const f32x4*>(init + at), up = *reinterpret_cast<const f32x4*>(init + at + 4);
#pragma unroll
          for (int j = 0; j < 4; j++) { a[j] = (E)lo[j]; a[4 + j] = (E)up[j]; }
        } else {
#pragma unroll
          for (int j = 0; j < 8; j++) a[j] = (E)init[lane + (uint32_t)((16 * kk + j) * D + 32 * t)];
        }
        acc[t] = mfma(a, xf[kk], acc[t]);
      }
    }
    if (!F16) {
      const float scale = exp2f(l2 * (float)max(rev ? n - 1 - r : r + 1, 0));
#pragma unroll
      for (int t = 0; t < NT; t++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[t][v] *= scale;
    }
  }
  // Decay of a score tile S^T[c][r] off the diagonal: a lane's factor times an element's, no exponent negative.
  // bf16: lambda^(|r - c|) of this lane's row and element v's key row, 32 positions apart, and one factor for the whole tiles in between.
  // fp16: what the scores carry when they are rounded may not take them below the type's range, which starts at 2^-14.  So
  // that is the decay to the tile's near edge only, and the sums, which then stand at that edge (`at`), take the rest in fp32.
  // And every row of a tile is scaled by a power of two (exponent `scaled` - 127, undone in the sums) that takes its largest
  // score to 2^14 or more (one of 2^-26 or more): the scores of small gradients one by one would be subnormal where their sum in
  // a state is not.  (Error against 64 bits, n 777, lambda 0.99, d 64, gradients of 1.2e-5: 1.9e-3 in the recurrence, 4.5e-3 with the
  // whole decay on the scores, 2.4e-3 without the scale, 1.7e-3 so.  Time, forward / backward, 16 chains of 777, d 128 14.2 -> 15.7,
  // 19.0 -> 20.2 us; d 64 9.8 -> 11.4, 11.5 -> 12.8.)
  const float lane_decay = exp2f(l2 * (float)(F16 ? (rev ? 4 * hh : 4 - 4 * hh) : rev ? 4 * hh - l32 + 32 : l32 - 4 * hh + 5));
  float od[16];
#pragma unroll
  for (int v = 0; v < 16; v++) od[v] = scalar_reg(exp2f(l2 * (float)(rev ? 8 * (v >> 2) + (v & 3) : 27 - 8 * (v >> 2) - (v & 3))));
  int at = rev ? n - 1 : -1, scaled = 127;
  auto rescale = [&](int gap, int now) __attribute__((always_inline)) {   // the sums, `gap` positions on
    const float f = fast_exp2(l2 * (float)max(gap, 0)) * __uint_as_float((uint32_t)(127 + now - scaled) << 23);
    scaled = now;
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[t][v] *= f;
  };

  for (int s = 0; s < nsteps; s++) {
    arrive(s);
    if (s + 1 < nsteps) issue(s + 1);
    const int tile = (step_first(s) >> 5) + kg;
    const int ahead = row0 + 32 * rh - 32 * tile;
    const int dist = rev ? -ahead : ahead;
    if (dist >= 0 && tile <= end_tile) {   // (wave-uniform: not a tile on the masked side)
      const E* const tY = sT[s & 1][0];
      const E* const tZ = sT[s & 1][1];
      f32x16 st = zero16();
#pragma unroll
      for (int ks = 0; ks < KS; ks++) st = mfma(la.read_row(tY, kg, ks), xf[ks], st);
      if (dist == 0) {
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int cc = 8 * (v >> 2) + 4 * hh + (v & 3);
          const int e = rev ? cc - l32 : l32 - cc;
          st[v] *= e >= 0 ? fast_exp2(l2 * (float)e) : 0.f;
        }
      } else {
        const float far = F16 ? lane_decay : lane_decay * fast_exp2(l2 * (float)(dist - 32));
#pragma unroll
        for (int v = 0; v < 16; v++) st[v] *= far * od[v];
      }
      if constexpr (F16) {
        float most = 0.f;
#pragma unroll
        for (int v = 0; v < 16; v++) most = fmaxf(most, fabsf(st[v]));
        const u32x2 halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(most), __float_as_uint(most), false, false);
        most = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));   // (the row's other keys)
        const int near = 32 * tile + (rev ? 0 : 31), to = dist == 0 ? r : near;
        rescale(rev ? at - to : to - at, min(max(127 + 14 - ((int)(__float_as_uint(most) >> 23) - 127), 127), 167));
        at = near;
        const float up = __uint_as_float((uint32_t)scaled << 23);
#pragma unroll
        for (int v = 0; v < 16; v++) st[v] *= up;
      }
      ex8<E> pf[2];
#pragma unroll
      for (int v = 0; v < 16; v++) pf[v >> 3][v & 7] = (E)st[v];
#pragma unroll
      for (int t = 0; t < NT; t++)
#pragma unroll
        for (int q = 0; q < 2; q++) acc[t] = mfma(la.read_cols(tZ, 32 * kg + 16 * q, t), pf[q], acc[t]);
    }
  }

  if constexpr (F16) rescale(kg == rh ? 0 : rev ? at - r : r - at, 127);   // (a group on the diagonal stands at its rows)

  // The key groups' sums: [group][row][feature], 16-byte pieces swizzled by the row.  Lane: position, elements 4 g .. + 3 of
  // tile t are value features 32 t + 8 g + 4 hh .. + 3.
  lds_barrier();   // the tiles are done with
  constexpr int PPR = D / 4;   // 16-byte pieces per row
  auto piece = [](int row, int c) { return row * D + 4 * (c ^ (row & (PPR - 1))); };
  float* const mine = part + kg * (kRows * D);
  const int groups = init != nullptr ? kGroups : min(kGroups, ntiles);   // those that have something to add
  if (kg < groups) {
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int g = 0; g < 4; g++)
        *reinterpret_cast<f32x4*>(mine + piece(32 * rh + l32, 8 * t + 2 * g + hh)) =
            f32x4{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
  }
  lds_barrier();
  constexpr int TPR = kWaves;      // threads per row
  constexpr int PPT = PPR / TPR;
  const int row = tid / TPR, c0 = (tid % TPR) * PPT;
  f32x4 o[PPT];
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < PPT; i++) {
    o[i] = *reinterpret_cast<const f32x4*>(part + piece(row, c0 + i));
#pragma unroll
    for (int g = 1; g < kGroups; g++)
      if (g < groups) o[i] += *reinterpret_cast<const f32x4*>(part + g * (kRows * D) + piece(row, c0 + i));
#pragma unroll
    for (int j = 0; j < 4; j++) sq = fmaf(o[i][j], o[i][j], sq);
  }
  if (NORM) {
#pragma unroll
    for (int m = 1; m < TPR; m <<= 1) sq += __shfl_xor(sq, m);
    const float rn = __builtin_amdgcn_rsqf(fmaf(sq, 1.f / (float)D, p.eps));
#pragma unroll
    for (int i = 0; i < PPT; i++) o[i] *= rn;
    if (tid % TPR == 0 && row0 + row < n) {
      const int64_t at = p.cu_seqlens != nullptr ? (int64_t)hi * p.rstd_stride + p.cu_seqlens[bi] : (int64_t)chain * p.rstd_stride;
      p.rstd[at + row0 + row] = rn;
    }
  }
  if (row0 + row < n) {
    void* const vw = which == 0 ? p.w[0] : which == 1 ? p.w[1] : p.w[2];
    E* const gw = reinterpret_cast<E*>(vw) + base + (int64_t)(row0 + row) * stride_n + 4 * c0;
#pragma unroll
    for (int i = 0; i < PPT; i += 2) {
      ex8<E> e8;
#pragma unroll
      for (int j = 0; j < 4; j++) { e8[j] = (E)o[i][j]; e8[4 + j] = (E)o[i + 1][j]; }
      *reinterpret_cast<ex8<E>*>(gw + 4 * i) = e8;
    }
  }
}

template <typename E, int D>
hipError_t launch(const ShortParams& p, hipStream_t s) {
  constexpr int head_dim_tiles = D / 32;
  const int64_t grid = (int64_t)p.batch * p.heads * ((int64_t)p.nscan * ((p.n + kRows - 1) / kRows) + (p.fin != nullptr ? head_dim_tiles * head_dim_tiles / kWaves : 0));
  if (grid == 0) return hipSuccess;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;   // (the rule that leads here keeps it far below)
  if (p.rstd != nullptr) hipLaunchKernelGGL((short_scan_kernel<E, D, true>), dim3((unsigned)grid), dim3(64 * kWaves), 0, s, p);
  else                   hipLaunchKernelGGL((short_scan_kernel<E, D, false>), dim3((unsigned)grid), dim3(64 * kWaves), 0, s, p);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_short_scans(int dtype, int head_dim, const ShortParams& p, hipStream_t s) {
  if (head_dim == 64) return dtype == kF16 ? launch<_Float16, 64>(p, s) : launch<__bf16, 64>(p, s);
  return dtype == kF16 ? launch<_Float16, 128>(p, s) : launch<__bf16, 128>(p, s);
}

}  // namespace la2

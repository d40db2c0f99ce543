// SDPA backward of one routing call for bf16 and D = 16 or 32 (App. A.5),
// with the route side resident in registers.
//
// A workgroup of eight waves owns one (batch, head), a window of route blocks
// (32 routes each) and a chunk of the N positions.  Its waves form RW route
// groups x PW = 8 / RW position groups; a wave keeps RB route blocks in
// registers for the whole launch (operands, their gradient accumulators and,
// in an encode, -L and -c as operands of one more product, below) and walks its
// position group's tiles of 32 positions.  The position-side
// rows of the next step are copied into LDS while the current one runs.
//
// "Query" is the side whose softmax row it is (routes in an encode,
// positions in the decode), "key" the other one.  Per 32 x 32 tile:
//   S' = Q K^T - L,  dP' = dOut V^T - c          (rows = queries, cols = keys)
//   P = 2^S',  dS = P dP'
//   key side    dV^T += dOut^T P,  dK^T += Q^T dS  (P, dS as they lie)
//   query side  dQ^T += K^T dS^T                   (dS transposed through LDS)
// so a tile needs one transpose only (2 KiB of the wave's own, read back by
// transposing LDS reads).  D = 16 takes its gradient products on
// v_mfma_f32_16x16x32 (no rows wasted on a 32-row tile of 16 channels); two
// v_permlane16_swap per register pair turn the 32 x 32 result into its two
// 16-column operands.
//
// -L and -c enter as three bf16 terms of one more K = 8 product (24 bits, all
// of an fp32 value's): as initial accumulators they took 32 registers per
// route block, and the freed ones hold twice the route blocks per wave, which
// halves the LDS traffic per tile.
//
// The route-side gradients stay in registers until the end of the chunk; the
// position-side ones are summed over the RW route groups through LDS, in a
// fixed order, one step later (so there is one barrier per step).
//
// What bounds it at D = 16: the vector pipe and the waits around it.  By shader
// counters at N = 2^20, M = 512, a tile of 32 positions times a route block costs
// a wave of an encode 88 vector instructions (16 of them exponentials at half
// rate, the sums over the route groups and the stores included), 458 clocks of
// the pipe, and 10 MFMAs; of the decode 78, 410 and 8.75.  The pipe is busy 0.66
// and 0.69 of the time, the matrix pipe 0.32 and 0.30; the rest is the barrier of
// a step (the older wave of a SIMD runs ahead and waits for the younger), the
// sum over the route groups and LDS bank conflicts (17 and 22 clocks).  At D = 32
// (2 x 50,000 x 256, M = 256: one tile per barrier) the pipe is busy 0.4 of the
// time and the waits are 0.3 to 0.4 of it.
// At N = 2^20, C = 128, H = 8, M = 512: decode 1.10 ms, encodes 1.22 and 1.26 ms
// (the second call's adds to a gradient, and its sums wait for the copies issued
// just before), against 3.29, 2.46 and 2.47 ms for the kernel that kept the
// positions in registers and walked the routes (it read every route operand per
// tile, added into a per-wave LDS slot per tile and needed two and four route
// windows there).  At 2 x 50,000 x 256, H = 8, M = 256 (D = 32): 116, 147 and 164 us
// against 418, 255 and 277.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "flarepp_device.hpp"
#include "flarepp_internal.hpp"
#include "flarepp_split.hpp"

namespace flarepp {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

__device__ __forceinline__ f32x16 mfma32(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// c + the row constants: a holds (hi, mid, lo, 0) per row, b ones in the first
// three of its k slots (lanes 0 .. 31)
__device__ __forceinline__ f32x16 mfma_rows(const s16x4& a, const s16x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, c, 0, 0, 0);
}
// k order of the operands made from a 32 x 32 result (lane row r4 = lane / 16,
// element j): of the 16-column operands after the swap, and of a transposed
// 16 x 16 pair.
__device__ __forceinline__ int swap_k(int r4, int j) { return 16 * (r4 & 1) + 8 * (j >> 2) + 4 * (r4 >> 1) + (j & 3); }
__device__ __forceinline__ int pair_k(int r4, int j) { return 16 * (j >> 2) + 4 * r4 + (j & 3); }

// Column of a transposed 16-column block that lane i of 16 holds.
__device__ __forceinline__ int perm16(int i) { return 8 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// Rows 0 .. 15 (a) and 16 .. 31 (b) of a 32 x 32 result, packed, become the
// operands of columns 0 .. 15 (a) and 16 .. 31 (b) with k order swap_k.
__device__ __forceinline__ void swap_cols(bf16x8& a, bf16x8& b) {
  u32x4 ua = __builtin_bit_cast(u32x4, a), ub = __builtin_bit_cast(u32x4, b);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(ua[i], ub[i], false, false);
    ua[i] = r[0];
    ub[i] = r[1];
  }
  a = __builtin_bit_cast(bf16x8, ua);
  b = __builtin_bit_cast(bf16x8, ub);
}

__device__ __forceinline__ bf16x8 pack8(const f32x4& a, const f32x4& b) {
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) { r[j] = (__bf16)a[j]; r[4 + j] = (__bf16)b[j]; }
  return r;
}
__device__ __forceinline__ bf16x8 pack8(const f32x16& a, int o) {
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = (__bf16)a[o + j];
  return r;
}

// Tiles per position group and step, and 16-byte pieces per tile and lane of
// the position-side gradients.
template <int D> constexpr int rs_pt() { return D == 16 ? 2 : 1; }
template <int D, bool DEC> constexpr int rs_pieces() { return (DEC ? 1 : 2) * (D == 16 ? 2 : 4); }
// Bytes: one stage (position rows of a step), one partial buffer.
constexpr int rs_stage_bytes(int D, bool dec, int rw) { return rs_positions(D, rw) * (4 * D + (dec ? 16 : 0)); }
// (one route group: the waves' 2 KiB scratch, over both buffers)
constexpr int rs_part_bytes(int D, bool dec, int rw) {
  return rw == 1 ? 8 * 1024 : 8 * (D == 16 ? 2 : 1) * (dec ? 1 : 2) * (D == 16 ? 2 : 4) * 1024;
}

template <int D, bool DEC, int RB>
__global__ __launch_bounds__(512) void k_attn_bwd_rs(AttnBwdRsParams p) {
  using T = __bf16;
  constexpr int KS = D / 16, PT = rs_pt<D>(), PIECES = rs_pieces<D, DEC>();
  constexpr int NK = D == 16 ? 1 : 2;   // k steps of a product over 32 routes or positions
  constexpr int NQF = D == 16 ? 2 : 4;  // f32x4 accumulators of a [D][32] product
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = lane_id(), g = lane >> 5, c = lane & 31, r4 = lane >> 4, i16 = lane & 15, wave = wave_id();
  const int RW = 1 << p.rw_log2, PW = 8 >> p.rw_log2, rw = wave & (RW - 1), pg = wave >> p.rw_log2;
  // the heads of one (batch, chunk) run on one XCD (workgroups are dealt to
  // the 8 XCDs in turn), so the token rows they share pieces of meet in its L2
  const int unit = (int)(blockIdx.x >> 3) / p.H * 8 + (blockIdx.x & 7), h = (int)(blockIdx.x >> 3) % p.H;
  if (unit >= p.B * p.R) return;  // whole workgroup, before any barrier
  const int b = unit / p.R, r = unit % p.R, bh = b * p.H + h;
  const int SP = PW * PT * 32;  // positions per step
  const int64_t pos0 = (int64_t)r * p.steps * SP;
  const int nsteps = (int)max((int64_t)0, min((int64_t)p.steps, (p.N - pos0 + SP - 1) / SP));

  const int stage_bytes = SP * (4 * D + (DEC ? 16 : 0));
  char* const stage = smem;
  f32x4* const parts = reinterpret_cast<f32x4*>(smem + 2 * stage_bytes);
  const int part_units = RW == 1 ? 0 : 8 * PT * PIECES * 64;

  const T* kx = static_cast<const T*>(p.k) + (int64_t)bh * p.N * D;
  const T* gx = DEC ? static_cast<const T*>(p.g) + (int64_t)b * p.g_sb + h * p.g_sh
                    : static_cast<const T*>(p.g) + (int64_t)bh * D * p.Np;

  // ---- position rows of step st into stage buffer st & 1 ----
  // K (and dY): per tile [D / 8 parts of 16 bytes][32 rows]; V (d-major):
  // per tile [D][32 positions]; decode: -L and -c of the positions.  Rows
  // past N repeat row N - 1.
  // (the lane index is re-read in the parts of a step that address memory, so
  // that their per-lane offsets do not stay in registers across the tiles)
  auto opaque = [](int x) __attribute__((always_inline)) {
    asm volatile("" : "+v"(x));
    return x;
  };
  auto stage_issue = [&](int st) __attribute__((always_inline)) {
    const int lane = opaque(lane_id()), c = lane & 31, g = lane >> 5;
    char* dst = stage + (st & 1) * stage_bytes;
    const int64_t n0 = pos0 + (int64_t)st * SP;
    const int nk = PW * PT * KS;
    for (int q = wave; q < 2 * nk; q += 8) {
      const bool second = q >= nk;
      const int u = second ? q - nk : q, tile = u / KS, sub = u % KS;
      const int64_t t0 = n0 + 32 * tile;
      const T* src;
      if (!DEC && second) {
        const int d = 16 * sub + (lane >> 2);
        src = gx + (int64_t)d * p.Np + min(t0 + 8 * (lane & 3), (int64_t)p.Np - 8);
      } else {
        const int64_t n = min(t0 + c, (int64_t)p.N - 1);
        src = (second ? gx + n * p.g_sn : kx + n * D) + 16 * sub + 8 * g;
      }
      lds_copy16(src, dst + q * 1024);
    }
    if constexpr (DEC) {
      // 16 bytes of every position: -L and -c as three bf16 terms each
      const char* src = static_cast<const char*>(p.lc) + (int64_t)bh * p.N * 16;
      for (int o = 64 * wave; o < SP; o += 512)
        if (o + lane < SP) lds_copy16(src + min(n0 + o + lane, (int64_t)p.N - 1) * 16, dst + 4 * SP * D + 16 * o);
    }
  };
  // The younger wave of a SIMD (w + 4), which sums the partials after its tiles
  // (below), goes first: by age the other one does and then waits for it at
  // the barrier.  Encode at D = 16 only (N = 2^20, M = 512: 1.37 -> 1.22 and
  // 1.48 -> 1.26 ms); the decode sums half as much and does not gain, D = 32
  // has one tile per barrier and loses 2%.
  if (D == 16 && !DEC && RW > 1 && wave >= 4) __builtin_amdgcn_s_setprio(1);
  if (nsteps > 0) stage_issue(0);

  // ---- route side, resident ----
  // encode: a, gr = rows of Q (scaled) and dOut, at, gt = their transposes
  // (k order swap_k, or the 32 x 32 one); decode: a, gr = rows of Q (scaled)
  // and Z, at = Q transposed (k order pair_k, or the 32 x 32 one)
  bf16x8 a[RB][KS], gr[RB][KS], at[RB][D == 16 ? 1 : 2], gt[RB][D == 16 ? 1 : 2];
  s16x4 nl[RB], nc[RB];  // encode: -L and -c of the block's routes
  f32x4 aq[RB][NQF], az[RB][NQF];  // dQ^T (both), dZ^T (decode)
  {
    // The window's rows of Q (scaled), Q and dOut or Z in bf16, and the
    // encode's -L and -c = -<dOut, Out>, through LDS behind the stages.
    // Routes past M: zero rows and no mass (encode: their P is zero); in the
    // decode, where they are softmax keys, the score rows repeat the last
    // route (P stays <= 1) and the product rows are zero.
    const int nr = 32 * RB * RW;
    T* const qs = reinterpret_cast<T*>(parts);
    T* const qb = qs + nr * D;
    T* const zb = qb + nr * D;
    float* const lc = reinterpret_cast<float*>(zb + nr * D);
    const int64_t zo = (int64_t)bh * p.M * D;
    auto rows = [&](const auto* q) __attribute__((always_inline)) {
      for (int t = threadIdx.x; t < nr * (D / 8); t += 512) {
        const int m = 32 * p.sb0 + t / (D / 8), d = 8 * (t % (D / 8));
        const int64_t o = (int64_t)min(m, p.M - 1) * D + d;
        const auto qv = load_frag(q + o);
        const f32x8 zv = load_frag(p.z + zo + o);
        const bool ok = m < p.M;
        bf16x8 x, y, z;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          x[j] = (T)(DEC || ok ? (float)qv[j] * p.sl2 : 0.f);
          y[j] = (T)(ok ? (float)qv[j] : 0.f);
          z[j] = (T)(DEC || ok ? zv[j] : 0.f);
        }
        *reinterpret_cast<bf16x8*>(qs + t * 8) = x;
        *reinterpret_cast<bf16x8*>(qb + t * 8) = y;
        *reinterpret_cast<bf16x8*>(zb + t * 8) = z;
      }
    };
    const int64_t qo = b * p.q_sb + h * p.q_sh;
    if (p.q_f32) rows(static_cast<const float*>(p.q) + qo);
    else rows(static_cast<const T*>(p.q) + qo);
    if constexpr (!DEC) {
      for (int t = threadIdx.x; t < nr; t += 512) {
        const int m = 32 * p.sb0 + t, mr = min(m, p.M - 1);
        float s = 0.f;
#pragma unroll
        for (int d = 0; d < D; d += 8) {
          const f32x8 x = load_frag(p.z + zo + (int64_t)mr * D + d), y = load_frag(p.out + zo + (int64_t)mr * D + d);
#pragma unroll
          for (int j = 0; j < 8; ++j) s += x[j] * y[j];
        }
        lc[t] = m < p.M ? -p.lse[(int64_t)bh * p.M + mr] * kLog2e : kNoMass;
        lc[nr + t] = m < p.M ? -s : 0.f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int m0 = 32 * (rw * RB + i);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        a[i][ks] = load_frag(qs + (m0 + c) * D + 16 * ks + 8 * g);
        gr[i][ks] = load_frag(zb + (m0 + c) * D + 16 * ks + 8 * g);
      }
#pragma unroll
      for (int kk = 0; kk < (D == 16 ? 1 : 2); ++kk)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int mk = m0 + (D == 16 ? (DEC ? pair_k(r4, j) : swap_k(r4, j)) : 16 * kk + acc_row16(g, j));
          const int d = D == 16 ? i16 : c;
          at[i][kk][j] = qb[mk * D + d];
          if (!DEC) gt[i][kk][j] = zb[mk * D + d];
        }
#pragma unroll
      for (int q = 0; q < NQF; ++q) {
        aq[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (DEC) az[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      if (!DEC) {
        // k slots 4 .. 7 (lanes 32 .. 63) are zero
        const s16x4 z = {0, 0, 0, 0};
        nl[i] = g ? z : split3(lc[m0 + c]);
        nc[i] = g ? z : split3(lc[nr + m0 + c]);
      }
    }
  }
  s16x4 ones;
#pragma unroll
  for (int j = 0; j < 4; ++j) ones[j] = (g == 0 && j < 3) ? (short)0x3f80 : (short)0;

  // Position-side results: runs of 8 channels, which = 0 the key gradient
  // (scaled by s), 1 the value gradient (encode).  n: position within the
  // step that starts at n0 (uniform).
  const int HD = p.H * D;
  auto emit = [&](int64_t n0, int n, int d, int which, f32x4 v0, f32x4 v1) __attribute__((always_inline)) {
    if (n >= p.N - n0) return;
    const int64_t base = ((int64_t)b * p.N + n0) * HD + h * D;  // uniform
    const int o = n * HD + d;
    T* const out = static_cast<T*>(which ? p.dg : p.dk) + base;
    if (!which) { v0 *= p.s; v1 *= p.s; }
    if (which ? p.acc_g : p.acc_k) {
      const bf16x8 old = load_frag(out + o);
#pragma unroll
      for (int q = 0; q < 4; ++q) { v0[q] += (float)old[q]; v1[q] += (float)old[4 + q]; }
      if (which && p.dg_lo) {
        const bf16x8 ol = load_frag(static_cast<const T*>(p.dg_lo) + base + o);
#pragma unroll
        for (int q = 0; q < 4; ++q) { v0[q] += (float)ol[q]; v1[q] += (float)ol[4 + q]; }
      }
    }
    const bf16x8 hi = pack8(v0, v1);
    *reinterpret_cast<bf16x8*>(out + o) = hi;
    if (which && p.dg_lo) {
#pragma unroll
      for (int q = 0; q < 4; ++q) { v0[q] -= (float)hi[q]; v1[q] -= (float)hi[4 + q]; }
      *reinterpret_cast<bf16x8*>(static_cast<T*>(p.dg_lo) + base + o) = pack8(v0, v1);
    }
  };
  // A tile's results lie in LDS as PIECES f32x4 per lane.  D = 16: pieces 2 w
  // and 2 w + 1 of lane l are channels 8 (l / 32) .. + 7 of position
  // 16 (l / 16 % 2) + l % 16 (after the swap below); D = 32: piece 4 w + a of
  // lane l is channels 8 a + 4 (l / 32) .. + 3 of position l % 32.

  // sum of step st's partials over the route groups, in order
  auto reduce = [&](int st) __attribute__((always_inline)) {
    const f32x4* pb = parts + (st & 1) * part_units;
    const int64_t n0 = pos0 + (int64_t)st * SP;
    const int units = PW * PT * PIECES * 32;
    for (int u = opaque(threadIdx.x); u < units; u += 512) {
      int l, q, tile, d, w, second;  // second: offset of the run's second half
      if constexpr (D == 16) {
        l = u & 63; q = (u >> 6) % (PIECES / 2) * 2; tile = (u >> 6) / (PIECES / 2);
        w = 16 * ((l >> 4) & 1); d = 8 * (l >> 5); second = RW * 64;
      } else {
        l = u & 31; q = (u >> 5) % PIECES; tile = (u >> 5) / PIECES;
        w = l & 16; d = 8 * (q & 3); second = 32;
      }
      const int n = w + (DEC ? perm16(l & 15) : (l & 15));
      const f32x4* x = pb + ((tile * PIECES + q) << p.rw_log2) * 64 + l;
      f32x4 s0 = x[0], s1 = x[second];
      for (int r = 1; r < RW; ++r) { s0 += x[r * 64]; s1 += x[r * 64 + second]; }
      emit(n0, 32 * tile + n, d, q / NQF, s0, s1);
    }
  };

  // ---- operands of a tile, from the staged rows ----
  struct Tile {
    bf16x8 kb[KS], gb[KS], kt[NK], yt[NK];
    s16x4 l, c;  // decode: -L and -c of the positions
  };
  // lane offsets (elements): rows as a score operand, rows transposed, and
  // the d-major V as a score operand
  const int row_off = (g * 32 + c) * 8;
  int tr_off0, tr_off1;  // elements 0 .. 3 and 4 .. 7
  {
    // rows row0 .. + 3 (lane i16 / 4 within them), channels 4 (i16 % 4) ..:
    // 16-byte part (i16 % 4) / 2 of a row (of its half r4 % 2 at D = 32)
    const int o = (((D == 16 ? 0 : 2 * (r4 & 1)) + ((i16 & 3) >> 1)) * 32 + (i16 >> 2)) * 8 + 4 * (i16 & 1);
    tr_off0 = o + 8 * (D == 16 ? (DEC ? swap_k(r4, 0) : pair_k(r4, 0)) : 4 * g);
    tr_off1 = o + 8 * (D == 16 ? (DEC ? swap_k(r4, 4) : pair_k(r4, 4)) : 8 + 4 * g);
  }
  const int v_off = (8 * g + (i16 >> 2)) * 32 + 16 * (r4 & 1) + 4 * (i16 & 3);
  auto load_tile = [&](Tile& t, int st, int tile) __attribute__((always_inline)) {
    const T* sk = reinterpret_cast<const T*>(stage + (st & 1) * stage_bytes) + tile * 32 * D;
    const T* sg = sk + SP * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      t.kb[ks] = load_frag(sk + row_off + ks * 512);
      if (DEC) t.gb[ks] = load_frag(sg + row_off + ks * 512);
      else t.gb[ks] = lds_tr_frag(sg + v_off + ks * 512, sg + v_off + ks * 512 + 128);
    }
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      t.kt[kk] = lds_tr_frag(sk + tr_off0 + kk * 128, sk + tr_off1 + kk * 128);
      if (DEC) t.yt[kk] = lds_tr_frag(sg + tr_off0 + kk * 128, sg + tr_off1 + kk * 128);
    }
    // A position past N repeats the last row.  Encode: its P is at most 1 and
    // its dS finite, and zero keys keep it out of dQ; decode: without mass its
    // P is zero.
    const int64_t left = p.N - (pos0 + (int64_t)st * SP + 32 * tile);  // uniform
    if (!DEC && left < 32) {
      int r = r4;
      asm volatile("" : "+v"(r));
#pragma unroll
      for (int kk = 0; kk < NK; ++kk)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if ((D == 16 ? pair_k(r, j) : 16 * kk + acc_row16(r >> 1, j)) >= left) t.kt[kk][j] = (T)0.f;
    }
    if (DEC) {
      typedef __attribute__((ext_vector_type(8))) short s16x8;
      const s16x8 x = *reinterpret_cast<const s16x8*>(sk + (2 * SP - tile * 32) * D + (32 * tile + c) * 8);
      t.l = s16x4{x[0], x[1], x[2], x[3]};
      t.c = s16x4{x[4], x[5], x[6], x[7]};
      if (left < 32 && c >= left) t.l = s16x4{split3(kNoMass)[0], 0, 0, 0};  // past N: no mass
    }
  };
  // dS^T: the lane's two runs of 8 queries' dS go to a 2 KiB scratch as rows
  // of 16 (one KiB per half), and come back transposed: lane i16 as column
  // perm16(i16), k order pair_k (D = 32: the 32 x 32 one).  The scratch is the
  // wave's own slot of this step's partials, written only after the tile.
  const int w_off = c * 16 + 8 * g;
  const int x_off = (i16 >> 2) * 16 + 4 * (i16 & 3) + 64 * (D == 16 ? r4 : g);

  // ---- a step: PT tiles x RB blocks of 32 routes, software pipelined ----
  // The score products of block k + 1 are issued as soon as block k has used
  // up its accumulators, and dS^T read back in block k is multiplied in block
  // k + 1, so neither the MFMA nor the LDS latency is waited out; the
  // scheduling barriers keep that order (the compiler's own order waits for
  // each product right after it).
  auto run_step = [&](int st) __attribute__((always_inline)) {
    constexpr int K = PT * RB;
    const int64_t n0 = pos0 + (int64_t)st * SP;
    Tile tl[PT];
    load_tile(tl[0], st, pg * PT);
    f32x16 s, dp;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto score = [&](int k) __attribute__((always_inline)) {
      const int i = k % RB;
      const Tile& t = tl[k / RB];
      s = mfma_rows(DEC ? t.l : nl[i], ones, zero16);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = DEC ? mfma32(t.kb[ks], a[i][ks], s) : mfma32(a[i][ks], t.kb[ks], s);
    };
    auto value = [&](int k) __attribute__((always_inline)) {
      const int i = k % RB;
      const Tile& t = tl[k / RB];
      dp = mfma_rows(DEC ? t.c : nc[i], ones, zero16);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) dp = DEC ? mfma32(t.gb[ks], gr[i][ks], dp) : mfma32(gr[i][ks], t.gb[ks], dp);
    };
    score(0);
    value(0);
    bf16x8 t0, t1;        // the previous block's dS^T
    f32x4 dk[NQF], dv[NQF];
    f32x16 dk32, dv32;
    auto zero_pos = [&]() __attribute__((always_inline)) {
      if constexpr (D == 16) {
#pragma unroll
        for (int q = 0; q < NQF; ++q) dk[q] = dv[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) dk32[e] = dv32[e] = 0.f;
      }
    };
    auto add16 = [&](f32x4 (&acc)[NQF], const bf16x8& a0, const bf16x8& b0, const bf16x8& a1, const bf16x8& b1)
        __attribute__((always_inline)) {
      f32x16 x;
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e] = acc[e >> 2][e & 3];
      x = mfma32(a0, b0, x);
      x = mfma32(a1, b1, x);
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e >> 2][e & 3] = x[e];
    };
    // the query side's product of block k
    auto query_side = [&](int k) __attribute__((always_inline)) {
      const int i = k % RB;
      const Tile& t = tl[k / RB];
      if constexpr (D == 16) {
        if (DEC) {
          dk[0] = mfma16(at[i][0], t0, dk[0]);
          dk[1] = mfma16(at[i][0], t1, dk[1]);
        } else {
          aq[i][0] = mfma16(t.kt[0], t0, aq[i][0]);
          aq[i][1] = mfma16(t.kt[0], t1, aq[i][1]);
        }
      } else if (DEC) {
        dk32 = mfma32(at[i][0], t0, dk32);
        dk32 = mfma32(at[i][1], t1, dk32);
      } else {
        add16(aq[i], t.kt[0], t0, t.kt[1], t1);
      }
    };
    // the position-side results of tile pt, to the partials or out
    auto flush = [&](int pt) __attribute__((always_inline)) {
      const int tile = pg * PT + pt;
      const int lane = opaque(lane_id()), g = lane >> 5, c = lane & 31, r4 = lane >> 4, i16 = lane & 15;
      if constexpr (D == 32) {
#pragma unroll
        for (int e = 0; e < 16; ++e) { dk[e >> 2][e & 3] = dk32[e]; dv[e >> 2][e & 3] = dv32[e]; }
      } else {
        // a lane's 4 channels of two positions -> 8 channels of one
        auto runs = [&](f32x4 (&x)[NQF]) __attribute__((always_inline)) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[0][e]), __float_as_uint(x[1][e]), false, false);
            x[0][e] = __uint_as_float(w[0]);
            x[1][e] = __uint_as_float(w[1]);
          }
        };
        runs(dk);
        if (!DEC) runs(dv);
      }
      if (RW == 1) {
        if constexpr (D == 16) {
          const int n = 32 * tile + 16 * (r4 & 1) + (DEC ? perm16(i16) : i16);
          emit(n0, n, 8 * g, 0, dk[0], dk[1]);
          if (!DEC) emit(n0, n, 8 * g, 1, dv[0], dv[1]);
        } else {
          // halves of the wave trade runs of 4 channels: rows 16 pr + 8 g .. + 7
          auto both = [&](const f32x4 (&x)[NQF], int which) __attribute__((always_inline)) {
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
              f32x4 v0, v1;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[2 * pr][e]), __float_as_uint(x[2 * pr + 1][e]), false, false);
                v0[e] = __uint_as_float(w[0]);
                v1[e] = __uint_as_float(w[1]);
              }
              emit(n0, 32 * tile + (DEC ? 16 * (r4 & 1) + perm16(i16) : c), 16 * pr + 8 * g, which, v0, v1);
            }
          };
          both(dk, 0);
          if (!DEC) both(dv, 1);
        }
      } else {
        f32x4* const slot = parts + (st & 1) * part_units + (((tile * PIECES) << p.rw_log2) + rw) * 64 + lane;
#pragma unroll
        for (int q = 0; q < PIECES; ++q) slot[(q << p.rw_log2) * 64] = q < NQF ? dk[q % NQF] : dv[q % NQF];
      }
    };
    zero_pos();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = k % RB, pt = k / RB;
      const Tile& t = tl[pt];
      // scratch: the wave's own slot of the tile's partials (written only
      // after the tile), or its own 2 KiB
      f32x4* const slot = RW == 1 ? parts + wave * 128 : parts + (st & 1) * part_units + ((((pg * PT + pt) * PIECES) << p.rw_log2) + rw) * 64;
      T* const x0 = reinterpret_cast<T*>(slot);
      T* const x1 = reinterpret_cast<T*>(slot + (RW == 1 ? 64 : RW * 64));
      __builtin_amdgcn_sched_barrier(0);
      if (k % RB == RB - 1 && pt + 1 < PT) load_tile(tl[pt + 1], st, pg * PT + pt + 1);
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = __builtin_amdgcn_exp2f(s[e]);
      bf16x8 p0 = pack8(s, 0), p1 = pack8(s, 8);
      __builtin_amdgcn_sched_barrier(0);
      if (k > 0 && i > 0) query_side(k - 1);  // (a tile's last one: below)
#pragma unroll
      for (int e = 0; e < 16; ++e) dp[e] *= s[e];
      __builtin_amdgcn_sched_barrier(0);
      if (k + 1 < K) score(k + 1);
      bf16x8 d0 = pack8(dp, 0), d1 = pack8(dp, 8);
      *reinterpret_cast<bf16x8*>(x0 + w_off) = d0;
      *reinterpret_cast<bf16x8*>(x1 + w_off) = d1;
      __builtin_amdgcn_sched_barrier(0);
      if (k + 1 < K) value(k + 1);
      if constexpr (D == 16) {
        t0 = lds_tr_frag(x0 + x_off, x0 + x_off + 256);
        t1 = lds_tr_frag(x1 + x_off, x1 + x_off + 256);
        swap_cols(p0, p1);
        swap_cols(d0, d1);
        if constexpr (DEC) {
          az[i][0] = mfma16(t.yt[0], p0, az[i][0]);
          az[i][1] = mfma16(t.yt[0], p1, az[i][1]);
          aq[i][0] = mfma16(t.kt[0], d0, aq[i][0]);
          aq[i][1] = mfma16(t.kt[0], d1, aq[i][1]);
        } else {
          dv[0] = mfma16(gt[i][0], p0, dv[0]);
          dv[1] = mfma16(gt[i][0], p1, dv[1]);
          dk[0] = mfma16(at[i][0], d0, dk[0]);
          dk[1] = mfma16(at[i][0], d1, dk[1]);
        }
      } else {
        // the half of the columns that this lane's row of 16 reads
        const T* xh = (r4 & 1) ? x1 : x0;
        t0 = lds_tr_frag(xh + x_off, xh + x_off + 128);
        t1 = lds_tr_frag(xh + x_off + 256, xh + x_off + 384);
        if constexpr (DEC) {
          add16(az[i], t.yt[0], p0, t.yt[1], p1);
          add16(aq[i], t.kt[0], d0, t.kt[1], d1);
        } else {
          dv32 = mfma32(gt[i][0], p0, dv32);
          dv32 = mfma32(gt[i][1], p1, dv32);
          dk32 = mfma32(at[i][0], d0, dk32);
          dk32 = mfma32(at[i][1], d1, dk32);
        }
      }
      if (i == RB - 1) {  // the tile's end
        query_side(k);
        flush(pt);
        if (k + 1 < K) zero_pos();
      }
    }
  };

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the first step's rows
  for (int st = 0; st < nsteps; ++st) {
    // this step's rows have landed (each wave has waited for its copies), the
    // last step's partials are complete and the buffers of the step before it
    // are free
    lds_barrier();
    if (st + 1 < nsteps) stage_issue(st + 1);
    // the two waves of a SIMD (w and w + 4) sum the last step's partials at
    // opposite ends of the step, so that one computes while the other waits
    // for LDS
    if (RW > 1 && st > 0 && wave < 4) reduce(st - 1);
    const bool full = pos0 + (int64_t)(st + 1) * SP <= p.N;  // uniform
    run_step(st);
    // wait for the copies, not for the stores issued after them (with one
    // route group a full step stores its results on every lane)
    constexpr int STORES = PT * (D == 16 ? 1 : 2);
    if (RW > 1 || !full) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(STORES * (DEC ? 1 : 2)) : "memory");
    if (RW > 1 && st > 0 && wave >= 4) reduce(st - 1);
  }
  __syncthreads();
  if (RW > 1 && nsteps > 0) reduce(nsteps - 1);
  __syncthreads();
  // route-side gradients: summed over the position groups in order, the
  // chunk's partial rows of this window ([m][d], padded to Mp)
  constexpr int RPC = (DEC ? 2 : 1) * NQF;  // pieces per block: dQ, then dZ
  f32x4* fin = reinterpret_cast<f32x4*>(smem);
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int q = 0; q < RPC; ++q)
      fin[(((rw * RB + i) * RPC + q) * PW + pg) * 64 + lane] = q < NQF ? aq[i][q % NQF] : az[i][q % NQF];
  __syncthreads();
  const int64_t po = ((int64_t)bh * p.R + r) * p.Mp * D + (int64_t)32 * p.sb0 * D;
  for (int u = threadIdx.x; u < p.nb * RPC * 64; u += 512) {
    const int l = u & 63, q = (u >> 6) % RPC, blk = (u >> 6) / RPC;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    for (int w = 0; w < PW; ++w) s += fin[((u >> 6) * PW + w) * 64 + l];
    const int col = DEC ? (l & 15) : perm16(l & 15);
    const int m = (D == 16 ? 16 * (q % NQF) : 16 * ((l >> 4) & 1)) + col, d = D == 16 ? 4 * (l >> 4) : 8 * (q % NQF) + 4 * (l >> 5);
    const int64_t o = po + (int64_t)(32 * blk + m) * D + d;
    if (q < NQF) store4(p.part_a + o, s[0] * p.s, s[1] * p.s, s[2] * p.s, s[3] * p.s);
    else store4(p.part_g + o, s[0], s[1], s[2], s[3]);
  }
}

template <int D, bool DEC, int RB>
hipError_t rs_go(const AttnBwdRsParams& p, hipStream_t s) {
  const int rw = 1 << p.rw_log2;
  const size_t fin = (size_t)8 * RB * (DEC ? 2 : 1) * (D == 16 ? 2 : 4) * 1024;
  const size_t lc = (size_t)32 * RB * rw * (6 * D + 8);  // the prologue's route rows, -L and -c
  const size_t lds = std::max<size_t>(2 * rs_stage_bytes(D, DEC, rw) + std::max<size_t>(2 * rs_part_bytes(D, DEC, rw), lc), fin);
  const void* fn = reinterpret_cast<const void*>(&k_attn_bwd_rs<D, DEC, RB>);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int64_t units = ((int64_t)p.B * p.R + 7) / 8 * 8;
  k_attn_bwd_rs<D, DEC, RB><<<(unsigned)(units * p.H), 512, lds, s>>>(p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bwd_rs(const AttnBwdRsParams& p, int D, bool dec, int rb, hipStream_t s) {
  if (D == 16) {
    if (rb == 4) return dec ? rs_go<16, true, 4>(p, s) : rs_go<16, false, 4>(p, s);
    if (rb == 2) return dec ? rs_go<16, true, 2>(p, s) : rs_go<16, false, 2>(p, s);
    return dec ? rs_go<16, true, 1>(p, s) : rs_go<16, false, 1>(p, s);
  }
  if (rb == 2) return dec ? rs_go<32, true, 2>(p, s) : rs_go<32, false, 2>(p, s);
  return dec ? rs_go<32, true, 1>(p, s) : rs_go<32, false, 1>(p, s);
}

}  // namespace flarepp

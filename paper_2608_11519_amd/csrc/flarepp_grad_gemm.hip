// The bf16 products of the mixer backward that reduce over tokens or over the
// four projections, for C = 64, 128 or 256.
//
// * k_wgrad: dW = A^T B over a chunk of the T tokens (A = X or Y, B a token
//   gradient), fp32 partials summed afterwards in a fixed order.  A token
//   contributes 4 C bytes and 2 C^2 operations, so the launch is bound by the
//   reads: rows go straight into a ring of LDS buffers several steps ahead
//   (about 100 KiB in flight per CU), and both operands, which need the tokens
//   as their k index, come out of the row-major tiles through transposing LDS
//   reads, with no register staging or repacking between.  2^20 x 128: 502 us
//   for nine arrays of 268 MB, X read by six problems (796 us with operand
//   tiles staged through registers); 100,000 x 256: 115 us (305; 164 with half
//   of the rows per workgroup, which read B twice).
// * k_rows_sum, k_rows_sum_stream: dX = sum_j G_j W_j^T over the four
//   projections by persistent workgroups.  2^20 x 128: 300 us for 1.6 GB (5.4
//   TB/s; 413 us as a tiled GEMM); 100,000 x 256: 87 us (172).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "flarepp_device.hpp"
#include "flarepp_internal.hpp"

namespace flarepp {
namespace {

using T = __bf16;

// ---------------------------------------------------------------------------
// weight gradients
// ---------------------------------------------------------------------------
// A workgroup computes the whole C x C product of its tokens; steps of 32
// tokens in a ring of NBUF LDS buffers ([32][C] of A, then of B).  Eight waves
// as 4 x 2 tiles of C / 4 x C / 2 (C = 64: 2 x 2 tiles of 32 x 32, twice: each
// half of the waves takes one half of a step's tokens).
template <int C> struct Wgrad {
  static constexpr int TI = C, TO = C;
  static constexpr int KG = C == 64 ? 2 : 1;              // groups of waves over a step's tokens
  static constexpr int WO = 2, WI = C == 64 ? 2 : 4;      // waves along o, i of one group
  static constexpr int NI = TI / WI / 32, NB = TO / WO / 32;  // 32 x 32 blocks of a wave
  static constexpr int BUF = 32 * (TI + TO) * 2;          // bytes of a step
  static constexpr int NBUF = C == 64 ? 12 : C == 128 ? 8 : 4;
  static constexpr int IPW = BUF / 1024 / 8;              // 1 KiB copies of a step per wave
  static_assert(WI * WO * KG == 8 && BUF % 8192 == 0 && BUF * NBUF <= 160 * 1024, "layout");
};

// LDS slot (16 bytes) of a row that holds its 16-byte chunk s: pairs of chunks
// are permuted by the row, so that the transposing reads of 8 rows fall in
// different banks (a 64-column row is half of the 256 bytes of banks)
template <int COLS>
__device__ __forceinline__ int wg_slot(int row, int s) {
  return s ^ (COLS == 64 ? 2 * ((row >> 1) & 3) : 2 * (row & 7));
}

template <int C>
__global__ __launch_bounds__(512) void k_wgrad(WgradParams p) {
  using W = Wgrad<C>;
  constexpr int TI = W::TI, TO = W::TO, NI = W::NI, NB = W::NB;
  __shared__ __attribute__((aligned(16))) char smem[W::BUF * W::NBUF];
  const int lane = lane_id(), g = lane >> 5, c = lane & 31, r4 = lane >> 4, i16 = lane & 15, wave = wave_id();
  // the problems of one token chunk run on one XCD (workgroups are dealt to
  // the 8 XCDs in turn), so X, which most of them read, comes from its L2
  // after the first read
  const int L = blockIdx.x, rr = L >> 3, prob = rr % p.nprob, chunk = rr / p.nprob * 8 + (L & 7);
  if (chunk >= p.nchunks) return;  // whole workgroup, before any barrier
  const int64_t t0 = (int64_t)chunk * p.chunk, t1 = min(p.T, t0 + p.chunk);
  const int nsteps = (int)((t1 - t0 + 31) / 32);
  const T* A = static_cast<const T*>(p.a[prob]);
  const T* B = static_cast<const T*>(p.b[prob]);

  // copies of step s: this wave's IPW KiB of the step's buffer (rows past the
  // end repeat the last one)
  auto issue = [&](int s) __attribute__((always_inline)) {
    if (s >= nsteps) return;
    char* dst = smem + s % W::NBUF * W::BUF;
#pragma unroll
    for (int q = 0; q < W::IPW; ++q) {
      const int u = wave * W::IPW + q;  // KiB of the buffer
      const bool isb = u >= TI / 16;
      const int cols = isb ? TO : TI, e = (isb ? u - TI / 16 : u) * 64 + lane;
      const int row = e / (cols / 8), slot = e % (cols / 8);
      const int ch = isb ? wg_slot<TO>(row, slot) : wg_slot<TI>(row, slot);
      const int64_t t = min(t0 + 32 * s + row, p.T - 1);
      lds_copy16((isb ? B : A) + t * C + 8 * ch, dst + u * 1024);
    }
  };
  for (int s = 0; s < W::NBUF - 1; ++s) issue(s);

  const int kg = wave / (W::WI * W::WO), wi = wave / W::WO % W::WI, wo = wave % W::WO;
  // k slots of a 16-token step: lanes 0 .. 31 rows 0 .. 3 and 8 .. 11, lanes
  // 32 .. 63 rows 4 .. 7 and 12 .. 15 (the same for both operands)
  const int row = 4 * g + (i16 >> 2);
  auto frag_off = [&](int cols, int f) __attribute__((always_inline)) {  // bytes, columns 32 f .. + 31
    const int s = 4 * f + 2 * (r4 & 1) + ((i16 & 3) >> 1);
    return row * cols * 2 + (cols == TO ? wg_slot<TO>(row, s) : wg_slot<TI>(row, s)) * 16 + 8 * (i16 & 1);
  };
  int aoff[NI], boff[NB];
#pragma unroll
  for (int f = 0; f < NI; ++f) aoff[f] = frag_off(TI, wi * NI + f);
#pragma unroll
  for (int f = 0; f < NB; ++f) boff[f] = 32 * TI * 2 + frag_off(TO, wo * NB + f);
  f32x16 acc[NI][NB];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int f = 0; f < NB; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][f][e] = 0.f;

  for (int s = 0; s < nsteps; ++s) {
    // step s has landed: at most the NBUF - 2 steps after it are in flight
    if (s + W::NBUF - 2 < nsteps) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(W::IPW * (W::NBUF - 2)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    issue(s + W::NBUF - 1);  // into the buffer of step s - 1, which every wave has left
    char* buf = smem + s % W::NBUF * W::BUF;
    const int left = (int)min((int64_t)32, t1 - t0 - 32 * s);
    if (left < 32) {  // the last rows: past the end they count as zero
      for (int e = threadIdx.x; e < W::BUF / 16; e += 512) {
        const int rw = e < 32 * TI / 8 ? e / (TI / 8) : (e - 32 * TI / 8) / (TO / 8);
        if (rw >= left) reinterpret_cast<f32x4*>(buf)[e] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < 2 / W::KG; ++k) {
      const int ks = W::KG == 2 ? kg : k;
      bf16x8 af[NI], bf[NB];
#pragma unroll
      for (int f = 0; f < NI; ++f) {
        const char* ap = buf + ks * 16 * TI * 2 + aoff[f];
        af[f] = lds_tr_frag(ap, ap + 8 * TI * 2);
      }
#pragma unroll
      for (int f = 0; f < NB; ++f) {
        const char* bp = buf + ks * 16 * TO * 2 + boff[f];
        bf[f] = lds_tr_frag(bp, bp + 8 * TO * 2);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int f = 0; f < NB; ++f) mma(acc[i][f], af[i], bf[f]);
    }
  }
  if constexpr (W::KG == 2) {
    // the second group's sums are added to the first's
    __syncthreads();
    float* x = reinterpret_cast<float*>(smem) + (wi * W::WO + wo) * 1024 + lane;
    if (kg == 1) {
#pragma unroll
      for (int e = 0; e < 16; ++e) x[64 * e] = acc[0][0][e];
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][0][e] += x[64 * e];
  }
  float* out = p.part + ((int64_t)prob * p.nchunks + chunk) * C * C + (int64_t)(32 * wi * NI) * C + 32 * wo * NB + c;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int f = 0; f < NB; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) out[(32 * i + acc_row(lane, e)) * C + 32 * f] = acc[i][f][e];
}

// out[o] = the sum, in order, of its problems' chunk partials; four values per
// thread, the loads of a group of eight partials issued before its adds
__global__ __launch_bounds__(256) void k_wgrad_sum(WgradSumParams p) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= (int64_t)p.nout * p.n) return;
  const int o = (int)(i / p.n);
  const int64_t e = i % p.n;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  for (int q = 0; q < 4 && p.prob[o][q] >= 0; ++q) {
    const float* x = p.part + (int64_t)p.prob[o][q] * p.nchunks * p.n + e;
    int r = 0;
    for (; r + 8 <= p.nchunks; r += 8) {
      f32x4 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const f32x4*>(x + (int64_t)(r + j) * p.n);
#pragma unroll
      for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; r < p.nchunks; ++r) s += *reinterpret_cast<const f32x4*>(x + (int64_t)r * p.n);
  }
  *reinterpret_cast<f32x4*>(p.out[o] + e) = s;
}

// ---------------------------------------------------------------------------
// input gradient
// ---------------------------------------------------------------------------
// C <= 128: the four weights' fragments stay in LDS (at most 128 KiB); eight
// waves, each walking tiles of 32 tokens with a tile's rows of one projection
// in registers while the next one's are loaded.
template <int KS>
__global__ __launch_bounds__(512) void k_rows_sum(RowsSumParams p) {
  constexpr int C = 16 * KS, NB = C / 32, SEG = C * C;  // output blocks, elements of a weight
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = lane_id(), g = lane >> 5, c = lane & 31, wave = wave_id();
#pragma unroll
  for (int j = 0; j < 4; ++j) copy_to_lds(p.wf[j], smem + j * SEG * 2, SEG / 8, 512);
  const T* wl = reinterpret_cast<const T*>(smem) + lane * 8;
  const int64_t tiles = (p.T + 31) / 32, stride = (int64_t)gridDim.x * 8;
  int64_t t = (int64_t)blockIdx.x * 8 + wave;
  auto load = [&](bf16x8 (&x)[KS], int64_t tile, int j) __attribute__((always_inline)) {
    const T* src = static_cast<const T*>(p.in[j]) + min(tile * 32 + c, p.T - 1) * C + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x[ks] = load_frag(src + 16 * ks);
  };
  bf16x8 xa[KS], xb[KS];
  if (t < tiles) load(xa, t, 0);
  lds_wait_barrier();
  f32x16 acc[NB];
  auto seg = [&](bf16x8 (&x)[KS], bf16x8 (&nx)[KS], int64_t tile, int j) __attribute__((always_inline)) {
    // this projection's rows are waited for first, then the next one's (or the
    // next tile's first) go out
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("; rows %0" : "+v"(x[ks]));
    if (j < 3) load(nx, tile, j + 1);
    else if (tile + stride < tiles) load(nx, tile + stride, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int q = 0; q < NB; ++q) mma(acc[q], x[ks], load_frag(wl + j * SEG + (q * KS + ks) * 512));
    // the LDS reads of k step ks + 1 go out ahead of the products of step ks
    __builtin_amdgcn_sched_group_barrier(0x100, NB, 0);
#pragma unroll
    for (int ks = 1; ks < KS; ++ks) {
      __builtin_amdgcn_sched_group_barrier(0x100, NB, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
  };
  for (; t < tiles; t += stride) {
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
    seg(xa, xb, t, 0);
    seg(xb, xa, t, 1);
    seg(xa, xb, t, 2);
    seg(xb, xa, t, 3);
    // rows = tokens, columns along the lanes: 128 contiguous bytes per row
    float* out = p.out + t * 32 * C + c;
    const int left = (int)min((int64_t)32, p.T - t * 32);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = acc_row(lane, e);
      if (row < left) {
#pragma unroll
        for (int q = 0; q < NB; ++q) out[row * C + 32 * q] = acc[q][e];
      }
    }
  }
}

// The same product at C = 256, where the four weights (512 KiB) do not fit in
// LDS: the tokens' rows do the waiting there instead.  A workgroup walks tiles
// of 64 tokens; each projection's rows [64][256] are one slot of a ring of
// four (direct copies, issued three slots ahead), and a wave computes 32 output
// columns for all 64 tokens with its weight fragments read from L2, which
// holds all four weights, one projection ahead.  Those are ordinary loads, and
// the compiler, which does not see the copies issued behind them, waits for
// them down to zero at the next step's start: a step's copies have one step to
// land, not three, and the counted wait ahead of the barrier only orders them.
// Every row is read once (100,000 tokens: 87 us for 307 MB; a quarter of the columns
// per workgroup with the weights in LDS read them four times: 138 us).
__global__ __launch_bounds__(512) void k_rows_sum_stream(RowsSumParams p) {
  constexpr int C = 256, KS = 16, TOK = 64, SLOT = TOK * C * 2, RING = 4;
  __shared__ __attribute__((aligned(16))) char smem[RING * SLOT];
  const int lane = lane_id(), g = lane >> 5, c = lane & 31, wave = wave_id();
  const int64_t tiles = (p.T + TOK - 1) / TOK;
  const int mine = (int)((tiles - blockIdx.x + gridDim.x - 1) / gridDim.x);  // this workgroup's tiles
  const int nseg = 4 * mine;
  // slot q of the sequence: projection q % 4 of tile q / 4; 16-byte chunk s of
  // a row lies at chunk s ^ (row % 8), so that a column of chunks falls in
  // different banks
  auto issue = [&](int q) __attribute__((always_inline)) {
    if (q >= nseg) return;
    const T* src = static_cast<const T*>(p.in[q & 3]);
    const int64_t t0 = (blockIdx.x + (int64_t)(q >> 2) * gridDim.x) * TOK;
    char* dst = smem + q % RING * SLOT;
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // 32 KiB, 4 copies of 1 KiB per wave (two rows each)
      const int k = 4 * wave + u, row = 2 * k + (ln >> 5);
      lds_copy16(src + min(t0 + row, p.T - 1) * C + 8 * ((ln & 31) ^ (row & 7)), dst + k * 1024);
    }
  };
  // this wave's weight fragments of projection j (output block = wave)
  // (the lane index is re-read in the loads and copies, so that their addresses
  // do not stay in registers across the tiles)
  auto weights = [&](bf16x8 (&w)[KS], int j) __attribute__((always_inline)) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const T* src = static_cast<const T*>(p.wf[j]) + (wave * KS * 64 + ln) * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) w[ks] = load_frag(src + ks * 512);
  };
  bf16x8 wa[KS], wb[KS];
  weights(wa, 0);
  for (int q = 0; q < RING - 1; ++q) issue(q);
  f32x16 acc[2];
  auto seg = [&](int q, bf16x8 (&w)[KS], bf16x8 (&nw)[KS]) __attribute__((always_inline)) {
    // slot q has landed: of the copies, at most those of the slots after it
    // are in flight (the weight loads and stores between them only make the
    // wait stricter)
    if (q + RING - 2 < nseg) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(4 * (RING - 2)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("; weights %0" : "+v"(w[ks]));
    if (q + 1 < nseg) weights(nw, (q + 1) & 3);
    asm volatile("" ::: "memory");  // the copies go out after the weight loads
    issue(q + RING - 1);            // into the slot of step q - 1, which every wave has left
    const char* slot = smem + q % RING * SLOT;
    // chunk (2 ks + g) ^ (c % 8): the low three bits repeat every four k steps
    const char* at[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) at[k] = slot + c * C * 2 + (((2 * k + g) ^ (c & 7)) << 4);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        mma(acc[h], load_frag(reinterpret_cast<const T*>(at[ks & 3] + (ks >> 2) * 128 + h * 32 * C * 2)), w[ks]);
    // the LDS reads of two k steps go out ahead of the products of the step
    // before them (all of them hoisted would not fit the registers)
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int ks = 0; ks < KS - 2; ks += 2) {
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
  };
  for (int m = 0; m < mine; ++m) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[h][e] = 0.f;
    seg(4 * m, wa, wb);
    seg(4 * m + 1, wb, wa);
    seg(4 * m + 2, wa, wb);
    seg(4 * m + 3, wb, wa);
    const int64_t t0 = (blockIdx.x + (int64_t)m * gridDim.x) * TOK;
    const int left = (int)min((int64_t)TOK, p.T - t0);
    float* out = p.out + t0 * C + 32 * wave + c;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = 32 * h + acc_row(lane, e);
        if (row < left) out[row * C] = acc[h][e];
      }
  }
}

template <int C>
hipError_t wgrad_go(const WgradParams& p, hipStream_t s) {
  k_wgrad<C><<<(unsigned)((p.nchunks + 7) / 8 * 8 * p.nprob), 512, 0, s>>>(p);
  return hipGetLastError();
}

template <int KS>
hipError_t rows_sum_go(const RowsSumParams& p, hipStream_t s) {
  constexpr size_t lds = (size_t)4 * 256 * KS * KS * 2;
  const void* fn = reinterpret_cast<const void*>(&k_rows_sum<KS>);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int64_t groups = ((p.T + 31) / 32 + 7) / 8;  // of eight tiles
  k_rows_sum<KS><<<(unsigned)std::min<int64_t>(groups, 256), 512, lds, s>>>(p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wgrad(const WgradParams& p, int C, hipStream_t s) {
  return C == 64 ? wgrad_go<64>(p, s) : C == 128 ? wgrad_go<128>(p, s) : wgrad_go<256>(p, s);
}

hipError_t launch_wgrad_sum(const WgradSumParams& p, hipStream_t s) {
  const int64_t n = (int64_t)p.nout * p.n / 4;
  k_wgrad_sum<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_rows_sum(const RowsSumParams& p, int C, hipStream_t s) {
  if (C == 256) {
    k_rows_sum_stream<<<(unsigned)std::min<int64_t>((p.T + 63) / 64, 256), 512, 0, s>>>(p);
    return hipGetLastError();
  }
  return C == 64 ? rows_sum_go<4>(p, s) : rows_sum_go<8>(p, s);
}

}  // namespace flarepp

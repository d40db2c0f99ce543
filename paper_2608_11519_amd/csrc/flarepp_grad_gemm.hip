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
//   tiles staged through registers); 100,000 x 256: 164 us (305).
// * k_rows_sum: dX = sum_j G_j W_j^T over the four projections, persistent
//   workgroups with the weights resident in LDS; a wave holds a tile's rows of
//   one projection in registers while the next one's are loaded.  2^20 x 128:
//   300 us for 1.6 GB (5.4 TB/s; 413 us as a tiled GEMM); 100,000 x 256: 138 us
//   (172), where four workgroups each read the rows for a quarter of the
//   columns.
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
// Workgroup tile TI x TO of C x C; steps of 32 tokens in a ring of NBUF LDS
// buffers ([32][TI] of A, then [32][TO] of B).  Eight waves as 4 x 2 tiles of
// 32 x TO / 2 (C = 64: 2 x 2 tiles of 32 x 32, twice: each half of the waves
// takes one half of a step's tokens).
template <int C> struct Wgrad {
  static constexpr int TI = C < 128 ? 64 : 128, TO = C;
  static constexpr int KG = C == 64 ? 2 : 1;              // groups of waves over a step's tokens
  static constexpr int WO = 2, WI = TI / 32;              // waves along o, i of one group
  static constexpr int NB = TO / WO / 32;                 // 32 x 32 blocks of a wave
  static constexpr int BUF = 32 * (TI + TO) * 2;          // bytes of a step
  static constexpr int NBUF = C == 64 ? 12 : C == 128 ? 8 : 5;
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
  constexpr int TI = W::TI, TO = W::TO, NB = W::NB;
  __shared__ __attribute__((aligned(16))) char smem[W::BUF * W::NBUF];
  const int lane = lane_id(), g = lane >> 5, c = lane & 31, r4 = lane >> 4, i16 = lane & 15, wave = wave_id();
  // the problems of one token chunk run on one XCD (workgroups are dealt to
  // the 8 XCDs in turn), so X, which most of them read, comes from its L2
  // after the first read
  constexpr int HALVES = C / TI;
  const int per = p.nprob * HALVES;
  const int L = blockIdx.x, rr = L >> 3, sub = rr % per, chunk = rr / per * 8 + (L & 7);
  if (chunk >= p.nchunks) return;  // whole workgroup, before any barrier
  const int prob = sub / HALVES, i0 = sub % HALVES * TI;
  const int64_t t0 = (int64_t)chunk * p.chunk, t1 = min(p.T, t0 + p.chunk);
  const int nsteps = (int)((t1 - t0 + 31) / 32);
  const T* A = static_cast<const T*>(p.a[prob]) + i0;
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
  const int aoff = frag_off(TI, wi);
  int boff[NB];
#pragma unroll
  for (int f = 0; f < NB; ++f) boff[f] = 32 * TI * 2 + frag_off(TO, wo * NB + f);
  f32x16 acc[NB];
#pragma unroll
  for (int f = 0; f < NB; ++f)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[f][e] = 0.f;

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
      const char* ap = buf + ks * 16 * TI * 2 + aoff;
      const bf16x8 af = lds_tr_frag(ap, ap + 8 * TI * 2);
      bf16x8 bf[NB];
#pragma unroll
      for (int f = 0; f < NB; ++f) {
        const char* bp = buf + ks * 16 * TO * 2 + boff[f];
        bf[f] = lds_tr_frag(bp, bp + 8 * TO * 2);
      }
#pragma unroll
      for (int f = 0; f < NB; ++f) mma(acc[f], af, bf[f]);
    }
  }
  if constexpr (W::KG == 2) {
    // the second group's sums are added to the first's
    __syncthreads();
    float* x = reinterpret_cast<float*>(smem) + (wi * W::WO + wo) * 1024 + lane;
    if (kg == 1) {
#pragma unroll
      for (int e = 0; e < 16; ++e) x[64 * e] = acc[0][e];
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] += x[64 * e];
  }
  float* out = p.part + ((int64_t)prob * p.nchunks + chunk) * C * C + (int64_t)(i0 + 32 * wi) * C + 32 * wo * NB + c;
#pragma unroll
  for (int f = 0; f < NB; ++f)
#pragma unroll
    for (int e = 0; e < 16; ++e) out[(int64_t)acc_row(lane, e) * C + 32 * f] = acc[f][e];
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
// Eight waves; a wave walks tiles of 32 tokens.  NB output blocks of 32
// columns per workgroup (C = 256: a quarter of them, the four quarters of one
// token stream on one XCD), so the four weights' fragments fill at most 128
// KiB of LDS.
template <int KS, int NB>
__global__ __launch_bounds__(512) void k_rows_sum(RowsSumParams p) {
  constexpr int C = 16 * KS, SL = C / 32 / NB, SEG = KS * NB * 512;  // slices, elements of a weight's slice
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = lane_id(), g = lane >> 5, c = lane & 31, wave = wave_id();
  const int L = blockIdx.x, rr = L >> 3, slice = rr % SL, stream = rr / SL * 8 + (L & 7);
  const int64_t streams = gridDim.x / SL;  // a multiple of 8
#pragma unroll
  for (int j = 0; j < 4; ++j)
    copy_to_lds(static_cast<const T*>(p.wf[j]) + (int64_t)slice * SEG, smem + j * SEG * 2, SEG / 8, 512);
  const T* wl = reinterpret_cast<const T*>(smem) + lane * 8;
  const int64_t tiles = (p.T + 31) / 32, stride = streams * 8;
  int64_t t = stream * 8 + wave;
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
    float* out = p.out + t * 32 * C + slice * NB * 32 + c;
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

template <int C>
hipError_t wgrad_go(const WgradParams& p, hipStream_t s) {
  const int per = p.nprob * (C / Wgrad<C>::TI);
  k_wgrad<C><<<(unsigned)((p.nchunks + 7) / 8 * 8 * per), 512, 0, s>>>(p);
  return hipGetLastError();
}

template <int KS, int NB>
hipError_t rows_sum_go(const RowsSumParams& p, hipStream_t s) {
  constexpr int SL = KS / 2 / NB;
  constexpr size_t lds = (size_t)4 * KS * NB * 1024;
  const void* fn = reinterpret_cast<const void*>(&k_rows_sum<KS, NB>);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // streams of 8 waves, a multiple of 8 (one XCD each), one workgroup per CU
  const int64_t tiles = (p.T + 31) / 32, want = ((tiles + 7) / 8 + 7) / 8 * 8;
  const int64_t streams = std::min<int64_t>(want, 256 / SL);
  k_rows_sum<KS, NB><<<(unsigned)(streams * SL), 512, lds, s>>>(p);
  return hipGetLastError();
}

}  // namespace

// Chunks of tokens: one round of workgroups over the 256 CUs, a multiple of 8
// (one XCD each) where there are that many, at least 128 tokens each.
int wgrad_chunks(int64_t T, int C, int nprob, int64_t* chunk) {
  const int64_t per = (int64_t)nprob * (C == 256 ? 2 : 1);
  int64_t n = std::max<int64_t>(1, 256 / per);
  if (n >= 8) n = n / 8 * 8;
  n = std::min(n, (T + 127) / 128);
  *chunk = ((T + n - 1) / n + 31) / 32 * 32;
  return (int)((T + *chunk - 1) / *chunk);
}

hipError_t launch_wgrad(const WgradParams& p, int C, hipStream_t s) {
  return C == 64 ? wgrad_go<64>(p, s) : C == 128 ? wgrad_go<128>(p, s) : wgrad_go<256>(p, s);
}

hipError_t launch_wgrad_sum(const WgradSumParams& p, hipStream_t s) {
  const int64_t n = (int64_t)p.nout * p.n / 4;
  k_wgrad_sum<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_rows_sum(const RowsSumParams& p, int C, hipStream_t s) {
  return C == 64 ? rows_sum_go<4, 2>(p, s) : C == 128 ? rows_sum_go<8, 4>(p, s) : rows_sum_go<16, 2>(p, s);
}

}  // namespace flarepp

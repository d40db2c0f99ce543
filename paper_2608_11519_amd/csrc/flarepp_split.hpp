// Work splits of the backward: which part of the positions, routes and tokens
// a workgroup takes.  Plain host C++ (no HIP), so that the rules can be
// compiled and checked by themselves.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace flarepp {

constexpr int kCUs = 256;

// ---- k_attn_bwd (fp32, and bf16 at D = 64) -----------------------------------
// LDS per wave: the short-side slot(s) [D][32 nsb + 4] fp32 (route index
// fastest, padded so that the lanes' rows fall in different banks) and one
// transpose tile [32][32 + 16 bytes] of T (dS, then P in the decode); per
// workgroup (encode) the routes' L and c.
constexpr size_t attn_bwd_tile_bytes(int elem_bytes) { return (size_t)32 * (32 + 16 / elem_bytes) * elem_bytes; }
constexpr size_t attn_bwd_wave_bytes(int D, int nsb, bool dec, int elem_bytes) {
  return sizeof(float) * (size_t)(dec ? 2 : 1) * D * (32 * nsb + 4) + attn_bwd_tile_bytes(elem_bytes);
}
// LDS of a launch over a window of nsb route blocks (Mp routes in all)
constexpr size_t attn_bwd_lds_bytes(int D, int nsb, int Mp, bool dec, int waves, int elem_bytes) {
  return (size_t)waves * attn_bwd_wave_bytes(D, nsb, dec, elem_bytes) + (dec ? 0 : 2 * sizeof(float) * (size_t)Mp);
}
constexpr int attn_bwd_waves(int D, int nsb, int Mp, bool dec, int elem_bytes) {
  for (int w = 4; w >= 1; w /= 2)
    if (attn_bwd_lds_bytes(D, nsb, Mp, dec, w, elem_bytes) <= 160 * 1024) return w;
  return 0;
}

// Over the long axis (keys of an encode, tokens of the decode): R chunks per
// (b, h) and tpw 32-position tiles per wave; over the routes: a launch covers
// nsb route blocks (a window) whose route-gradient slots fit the LDS budget at
// four waves; the windows run one after another.
struct BwdSplit {
  int waves, R, tpw, nsb;
};

// Time of R chunks per (b, h), in tiles of one wave: the kernel's registers
// hold one workgroup per CU, so the workgroups run in rounds of 256, each as
// long as a wave's tiles and a quarter of a tile for its prologue and partials.
constexpr double bwd_rounds_time(int64_t BH, int64_t tiles, int64_t waves, int64_t R) {
  const int64_t tpw = (tiles + R * waves - 1) / (R * waves);
  return (double)((BH * R + kCUs - 1) / kCUs) * ((double)tpw + 0.25);
}

// The chunk count, up to two rounds of workgroups' worth, that takes the least
// time (the fewest chunks of equal ones): a count a little over a whole round
// leaves another one nearly empty (1 x 20,011 tokens, M = 100, D = 16, fp32: 316
// workgroups 64, 59 and 56 us, 212 47, 44 and 42), a count that must fit one
// round leaves CUs idle with more than 128 pairs (160 pairs of 3,000 tokens,
// M = 64, decode: 160 workgroups 181 us in fp32 at D = 16 and 298 in bf16 at D = 64,
// 480 workgroups 132 and 219).
inline BwdSplit bwd_split(int64_t BH, int64_t Nl, int D, int Mp, bool dec, int elem_bytes, size_t budget) {
  BwdSplit sp{};
  const int NS = Mp / 32;
  int nwin = 1;
  while (nwin < NS && attn_bwd_lds_bytes(D, (NS + nwin - 1) / nwin, Mp, dec, 4, elem_bytes) > budget) ++nwin;
  sp.nsb = (NS + nwin - 1) / nwin;
  sp.waves = attn_bwd_waves(D, sp.nsb, Mp, dec, elem_bytes);
  const int64_t tiles = (Nl + 31) / 32, W = sp.waves;
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>((2 * kCUs + BH - 1) / BH, (tiles + W - 1) / W));
  int64_t R = 1;
  for (int64_t r = 2; r <= most; ++r)
    if (bwd_rounds_time(BH, tiles, W, r) < bwd_rounds_time(BH, tiles, W, R)) R = r;
  const int64_t tpw = (tiles + R * W - 1) / (R * W);
  sp.R = (int)((tiles + tpw * W - 1) / (tpw * W));
  sp.tpw = (int)tpw;
  return sp;
}

// ---- k_attn_bwd_rs (bf16, D = 16 or 32) ----------------------------------------
struct RsSplit {
  int rb, rw_log2, nbw;  // route blocks per wave, log2 route groups, route blocks per launch
  int R, steps;          // chunks per (b, h), steps of rs_positions positions per chunk
};
constexpr int rs_positions(int D, int rw) { return (8 / rw) * (D == 16 ? 2 : 1) * 32; }

inline RsSplit rs_split(int64_t B, int64_t H, int64_t N, int D, int Mp) {
  RsSplit sp{};
  sp.rb = 1;
  const int NS = Mp / 32;
  // route blocks per wave: what the registers hold next to the tile's work
  const int cap = D == 16 ? 4 : 2;
  while (sp.rb < cap && sp.rb < NS) sp.rb *= 2;
  // route groups: the fewest (a power of two) that hold the routes, at most 8
  while (sp.rw_log2 < 3 && (sp.rb << sp.rw_log2) < NS) ++sp.rw_log2;
  sp.nbw = sp.rb << sp.rw_log2;
  const int64_t SP = rs_positions(D, 1 << sp.rw_log2), steps = (N + SP - 1) / SP, BH = B * H;
  // chunks: one workgroup per CU; with more (b, h) pairs than CUs, the count
  // whose last round of workgroups is fullest
  int64_t R = std::max<int64_t>(1, kCUs / BH);
  if (BH > kCUs / 2) {
    double best = 1e30;
    for (int64_t x = 1; x <= 4; ++x) {
      const double t = (double)((BH * x + kCUs - 1) / kCUs) / (double)x * (1.0 + 0.02 * (double)x);
      if (t < best) { best = t; R = x; }
    }
  }
  R = std::min(R, steps);
  sp.steps = (int)((steps + R - 1) / R);
  sp.R = (int)((steps + sp.steps - 1) / sp.steps);
  return sp;
}

// ---- k_wgrad ---------------------------------------------------------------------
// Chunks of tokens: one round of workgroups over the CUs, a multiple of 8 (one
// XCD each) where there are that many, at least 128 tokens each.
inline int wgrad_chunks(int64_t T, int nprob, int64_t* chunk) {
  int64_t n = std::max<int64_t>(1, kCUs / nprob);
  if (n >= 8) n = n / 8 * 8;
  n = std::min(n, (T + 127) / 128);
  *chunk = ((T + n - 1) / n + 31) / 32 * 32;
  return (int)((T + *chunk - 1) / *chunk);
}

}  // namespace flarepp

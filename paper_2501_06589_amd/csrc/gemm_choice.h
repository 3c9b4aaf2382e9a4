// Which tile shape and split of K the packed-weight GEMM takes (host only, no HIP: gemm_duo_kernel, gemm_lds_kernel and gemm_ring_kernel are in
// prefill_kernels.hip).
#pragma once

#include <math.h>

struct GemmShape { int M, N, K, ldx, epilogue, n_peers; };   // as in GemmArgs

// Tile shapes of the kernels and what a stage of 64 k takes of a workgroup (us).  Ring tiles (one workgroup per CU): on a full
// chip, and the share of that on a nearly empty one.  Duo tiles (two per CU): with every CU holding two; the share of that where
// few CUs hold two (two); where every CU holds one (one), or few do (alone).
enum { TILE_64x64, TILE_64x128, TILE_128x64, TILE_128x128, TILE_128x256, TILE_256x256, TILE_DUO_128, TILE_DUO_192, TILE_DUO_256, TILE_COUNT };
static const struct { int bm, bn; float stage_us, alone, one, two; } gemm_tiles[TILE_COUNT] = {
    {64, 64, 0.24f, 1.0f, 0, 0},    {64, 128, 0.39f, 1.0f, 0, 0},   {128, 64, 0.35f, 0.87f, 0, 0},
    {128, 128, 0.58f, 0.82f, 0, 0}, {128, 256, 0.99f, 0.85f, 0, 0}, {256, 256, 1.59f, 0.74f, 0, 0},
    {128, 128, 0.888f, 0.435f, 0.52f, 0.964f}, {128, 192, 1.316f, 0.418f, 0.50f, 0.814f}, {128, 256, 1.659f, 0.419f, 0.501f, 0.808f}};

// Estimated time (us) of a tile shape and split on the whole chip (256 CUs, which the fit is made on): the rounds of workgroups
// (start: a workgroup's start and end) against one pass over the weights, and the partial products of a split.  Ring tiles: the larger
// of the two, fitted to 3900 measured times (the projections of the 1.2B, 8B and 70B R = 8 / R = 4 shapes at 17 - 6000 rows, every
// tile, splits 1 - 8; rms error 7 %).  Duo tiles: the root of the sum of their squares, fitted to 1900 measured times (the same
// shapes at 80 - 8192 rows; rms error 8 %).  What it picks is on average 1.2 % off the fastest measured tile and split at 257 - 1024 rows and 0.6 % above, at worst
// 18 %.  (Sums of squares with refitted constants for the ring tiles too: 0.6 instead of 5.7 % off at up to 64 rows measured alone, but
// their larger tiles and splits leave less to the kernels beside: 8B shape, decode of 64 sequences 2981 -> 3277 us.)
// The products alone were measured: the bytes of a residual epilogue (epilogue 3: 26 per element with seven peers and a copy,
// 180 us at 4001 x 8192) are not in it, so there it chooses by the smaller part of the launch where K is short.
inline float gemm_cost(int tile, int M, int N, int K, int ksplit) {
  const auto& t = gemm_tiles[tile];
  const bool duo = tile >= TILE_DUO_128;
  const int slots = duo ? 512 : 256;
  const long wgs = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * ksplit;
  const int stages = (K + 63) / 64, per = (stages + ksplit - 1) / ksplit;
  const float last = (float)(wgs % slots) / (float)slots;
  const float start = duo ? 6.4f : 2.6f;
  float tiles_us = (float)(wgs / slots) * (start + (float)per * t.stage_us);
  if (last > 0.f) {
    const float share = !duo ? t.alone + (1.f - t.alone) * last
                        : last <= 0.5f ? t.alone + (t.one - t.alone) * 2.f * last : t.two + (1.f - t.two) * (2.f * last - 1.f);
    tiles_us += start + (float)per * t.stage_us * share;
  }
  const float weights = (float)N * (float)K * 2.0f, parts = ksplit > 1 ? (float)ksplit * (float)M * (float)N * 8.0f : 0.f;
  if (duo) {
    const float mem_us = 1.6f + weights / 6.07e6f;
    return sqrtf(tiles_us * tiles_us + mem_us * mem_us) + parts / 7.1e6f;
  }
  const float mem_us = 3.4f + weights / 6.3e6f;
  return (tiles_us > mem_us ? tiles_us : mem_us) + parts / 6.0e6f;
}

// gemm_duo_kernel's requests have 32-bit byte offsets: 128 rows of the activations, jt packed tiles side by side
inline bool gemm_duo_reaches(int ldx, int K, int jt) {
  return (long long)ldx * 256 + (long long)K * 2 <= 0x7fffffffll && (long long)K * 32 * jt <= 0x7fffffffll;
}

// Which of the 256 x 256 and the duo tiles: where both epilogues are cheap the model's; a SwiGLU epilogue costs a 256 x 256 round, which
// nothing hides, 7 us (8192 x 28672 x 4096 in place 1561 us, duo 1469; but 400 rows, one round, 111 against 125), and peers rule it out
// (O of the 70B R = 4 shard, 32768 rows: 1450 against 1330).  Without peers its residual update is the faster one where it fills the
// chip (8B shape, 8192 rows, O + down: 962 against 1030 us in place).
inline int gemm_best_tile(const GemmShape& a, int ksplit, float* cost) {
  const int M = a.M, N = a.N, K = a.K;
  int best = -1;
  float best_us = 0.f;
  for (int t = 0; t < TILE_COUNT; ++t) {
    if (t == TILE_256x256 && (ksplit > 1 || (K & 63) || K < 256)) continue;                   // (what gemm_lds_kernel takes)
    if (t == TILE_256x256 && (a.epilogue == 3 ? a.n_peers > 0 : a.epilogue == 1 && M > 1024)) continue;
    // duo tiles: from 257 rows on (below, the ring's deeper queue of weights is faster: 200 x 7168 x 8192 38 against 45 us)
    if (t >= TILE_DUO_128 && (M <= 256 || (K & 63) || !gemm_duo_reaches(a.ldx, K, gemm_tiles[t].bn / 64))) continue;
    if (t == TILE_64x64 && a.epilogue == 3) continue;   // (16 columns per wavefront: more sums of squares per row than the buffer holds)
    float us = gemm_cost(t, M, N, K, ksplit);
    if (t == TILE_256x256 && a.epilogue == 1) us += 7.0f * (float)(((long)((M + 255) / 256) * ((N + 255) / 256) + 255) / 256);
    if (best < 0 || us < best_us) { best = t; best_us = us; }
  }
  if (cost) *cost = best_us;
  return best;
}

// epilogue 0: the number of workgroups along K that suits the product (see gemm_ksplit)
inline int gemm_best_split(int M, int N, int K, int max_split, float extra_us) {
  const int stages = (K + 63) / 64;
  const GemmShape a{M, N, K, K, 0, 0};
  int best = 1;
  float best_us = 0.f;
  gemm_best_tile(a, 1, &best_us);
  for (int ks = 2; ks <= max_split && ks <= 16; ++ks) {
    const int per = (stages + ks - 1) / ks;
    if ((stages + per - 1) / per != ks) continue;   // (a split would be left without work)
    float us;
    gemm_best_tile(a, ks, &us);
    us += extra_us;
    if (us < best_us) { best = ks; best_us = us; }
  }
  return best;
}

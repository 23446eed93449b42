// Tile and split-K planning shared by the dense and MoE FFN launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include "gemm.h"

namespace aflex {

// Output columns per gate/up tile (x2 weight rows) and per down tile. The tiles
// of 128 rows and more take a CU's whole LDS (one work-group per CU).
inline int gate_bn(int bm) { return bm >= 128 ? 128 : 64; }

inline int down_bn(int bm) { return bm >= 128 ? 256 : 128; }
// Work-groups the down GEMM's split-K aims for: one round of the chip for the
// tiles of one work-group per CU; smaller tiles run two per CU.
constexpr int kOneWgPerCuTarget = 256;
inline int down_target(int bm) { return bm >= 128 ? kOneWgPerCuTarget : (bm == 64 ? 2048 : 512); }
// Work-groups resident on the 256 CUs at once: one per CU for the tiles of 128
// rows and more (the whole LDS), two for the smaller ones.
inline int concurrent_wgs(int bm) { return bm >= 128 ? 256 : 512; }

struct FfnPlan {
  int bm;           // rows per m-tile: 32, 64, 128 or 256
  bool nt;          // weight loads are non-temporal
  int down_splits;  // split-K factor of the down GEMM
  int down_kps;     // k elements per split (multiple of 64)
};

// Rows per m-tile for grouped GEMMs with the given average rows per expert.
// Up to 32 rows a tile covers a typical expert (its weights are streamed once);
// up to 48 rows 64-row tiles, two work-groups per CU, up to 96 rows the 8-wave
// 128-row tile; beyond, the 256-row shape, which holds an expert of up to 256 rows
// in one tile where more and more experts take two of 128. Mixtral shapes, 32
// rows per expert: 481 us with 64-row tiles, 460 with 128; 47: 505 and 474; 60: 547
// and 481 (for experts with few column tiles plan_moe goes back to 64); 80 rows: 508
// us with 128-row tiles, 508 with 256; 95: 519 and 518; 112: 613 and 532; 127: 674
// and 552; 144: 818 and 565.
//
// An expert's rows are split evenly over its row tiles (tile_rows below), so
// one just over a multiple of 256 rows has no nearly empty tile that streams all
// of its weights for a few rows.
inline int pick_bm(double rows_per_expert) {
  if (rows_per_expert * 1.3 <= 32) return 32;
  if (rows_per_expert <= 48) return 64;
  if (rows_per_expert <= 96) return 128;
  return 256;
}

// Rows per tile when n rows take the fewest tiles of at most bm rows: even
// shares, in whole 32-row blocks, for the 256-row tiles, which multiply only
// filled blocks (Mixtral T = 2048, 472-541 rows per expert: 192 + 192 + 157
// instead of 256 + 256 + 29); else bm.
__host__ __device__ inline int tile_rows(int n, int bm) {
  if (bm != 256 || n <= bm) return bm;
  const int tiles = (n + bm - 1) / bm, blocks = (n + 31) / 32;
  return (blocks + tiles - 1) / tiles * 32;
}

// Split K of the down GEMM, keeping at least `min_steps` 64-wide k-steps per
// split. With `slots` > 0 (the tile count is exact: dense GEMMs, and the
// one-work-group-per-CU tiles) the split count is the smallest whose
// work-groups fill the rounds of `slots` concurrent work-groups they need to
// at least 90% (measured best for the dense down GEMM at T = 256 ... 4096:
// 12, 6, 3, 3-4 splits; a nearly empty last round leaves a few work-groups
// streaming alone at the end); more splits only add fp32 partials to reduce.
// Otherwise (a worst-case tile count) about `target` work-groups.
inline void plan_splits(int base_tiles, int K, int target, int slots, int min_steps, int* splits, int* kps) {
  const int ksteps = K / 64;
  int smax = ksteps / min_steps;
  if (smax < 1) smax = 1;
  int s = (target + base_tiles - 1) / base_tiles;
  if (slots > 0) {
    double best_u = 0.0;
    for (int c = 1; c <= smax && c <= 64; ++c) {
      const long long wgs = (long long)base_tiles * c;
      const double u = (double)wgs / (double)(((wgs + slots - 1) / slots) * slots);
      if (u >= 0.9) {
        s = c;
        break;
      }
      if (u > best_u + 1e-9) {
        best_u = u;
        s = c;
      }
    }
  }
  if (s > smax) s = smax;
  if (s < 1) s = 1;
  const int steps = (ksteps + s - 1) / s;
  *splits = (ksteps + steps - 1) / steps;
  *kps = steps * 64;
}

// Weights up to this size load ordinarily, larger ones, where each byte is read
// by one work-group, non-temporally. The small ones may still be in the 256 MB
// Infinity Cache when a next call needs them (the other microbatches of a layer, a
// small model), and lose nothing where they are not. Times in us, ordinary and
// non-temporal loads, with the weights rotated through 1.3 GB and repeated:
//                                    rotated        repeated
//   linear 8192 x 5120 (84 MB), T = 64   26.6  28.6   22.4  28.5
//   linear 8192 x 5120, T = 32           23.6  24.3   19.4  23.2
//   SwiGLU 2816 x 9216 (156 MB), T = 64  51.3  53.6   39.0  53.5
//   SwiGLU 4096 x 14336 (352 MB), T = 32 76.2  74.1   83.8  82.0
constexpr long long kKeepWeightBytes = 160ll << 20;
// The same line up to 16 tokens, and for the experts of a MoE call, where rotated
// weights stream faster non-temporally from smaller sizes on:
//   linear 5120 x 5120 (52 MB), T = 8    17.4  17.2   13.9  15.4
//   linear 8192 x 5120 (84 MB), T = 8    21.7  20.7   17.9  18.9
//   SwiGLU 2048 x 4096 (50 MB), T = 8    24.2  24.3   19.7  22.8
//   MoE E = 8, 2048 x 768 (75 MB), T = 24    33.5  32.9   27.2  31.8
//   MoE E = 8, 1024 x 2816 (138 MB), T = 24  43.6  41.3   34.3  39.8
constexpr long long kKeepFewRowsBytes = 48ll << 20;

// Work-groups of a GEMM below which smaller tiles, of which there are more, are
// faster although they read more (256 CUs). SwiGLU 4096 x 14336, 128-row tiles
// (112 work-groups) and 64-row tiles: T = 40 86 and 71 us; 256- (112) and 128-row
// tiles: T = 256 145 and 124 us. 5120 x 25600 (200 work-groups): T = 40 143 and
// 157 us; 2048 x 22400 (175): T = 200 91 and 113 us.
constexpr int kFewWorkGroups = 160;
// The same for MoE calls, whose tile count is an estimate (every expert the
// average): so few that tiles of half the height still fit one round when the
// estimate is off. E = 8, 512 x 512, k = 2, T = 1000: 54.7 us with 256-row tiles, 31.7
// with 64; E = 4, 1024 x 1024, T = 300: 48.4 and 31.2; with 144 work-groups of 256
// rows (E = 3, 4096 x 3008, k = 1, T = 1000) 127 us, with 128 rows 128. The line is not
// tight: E = 2, 2048 x 4096, k = 1, T = 300, 128 work-groups of 128 rows, 64.7, with 64
// rows 58.8.
constexpr int kFewGroupedWorkGroups = 112;

// Tiles of a MoE call. `once`: experts' rows are expected to fit one tile (average
// rows per expert x 1.3 <= bm, the margin pick_bm uses for 32-row tiles; always at
// 32 rows), so each expert's weights are streamed once and, where they are more
// than stays cached, load non-temporally (4-5% faster at 32-48 rows per expert on
// 64-row tiles, 11% at 64 on 128-row tiles, 5-6% at 112-190 on 256-row tiles:
// T = 509 580 -> 550 us).
struct MoePlan {
  int bm;  // rows per m-tile: 32, 64, 128, 256 or 320
  bool once, nt;
};

// Row tiles of 256 that E experts are expected to take, their row counts spread
// normally about the average.
inline double expected_tiles256(int E, double avg, double sigma) {
  double t = E;
  for (int j = 1; 256.0 * j < avg + 6.0 * sigma + 1.0; ++j)
    t += sigma > 0.0 ? E * 0.5 * erfc((256.0 * j - avg) / (sigma * sqrt(2.0))) : (avg > 256.0 * j ? E : 0);
  return t;
}

// `k` experts per token. Where enough experts are expected to take one more
// 256-row tile for the gate/up GEMM to need a second round of the chip, and
// 320-row tiles (the eight-wave kernel, ten row blocks) hold them in one, those
// are faster although their loop is not (256 rows -> 320): E = 8, k = 2, 1024 x
// 3584, T = 1000 110.7 -> 101.9 us; 4096 x 3584, T = 1060 277 -> 259; E = 4, k = 2,
// 3072 x 4096, T = 1120 223 -> 204. With rounds to spare they are not (E = 8, k = 2,
// 4096 x 14336, T = 1000: 849 and 934), nor where the 256-row ones fit one (E = 8,
// k = 2, 512 x 4096, T = 968: 77 and 81).
inline MoePlan plan_moe(long long pairs, int H, int I, int E, int k) {
  MoePlan pl;
  const double rows = (double)pairs / E;
  pl.bm = pick_bm(rows);
  const long long avg = (pairs + E - 1) / E;
  auto work_groups = [&](int bm) { return E * ((avg + bm - 1) / bm) * ((I + gate_bn(bm) - 1) / gate_bn(bm)); };
  while (pl.bm > 64 && work_groups(pl.bm) <= kFewGroupedWorkGroups) pl.bm /= 2;
  if (pl.bm == 256) {
    const int ntiles = (I + gate_bn(256) - 1) / gate_bn(256), round = concurrent_wgs(256);
    const double sigma = sqrt(rows * (1.0 - (double)k / E));  // tokens choose independently
    if (E * ceil((rows + 3.0 * sigma) / 320.0) * ntiles <= round &&
        floor(expected_tiles256(E, rows, sigma) + 0.5) * ntiles > round)
      pl.bm = 320;
  }
  pl.once = pl.bm == 32 || (pl.bm != 320 && rows * 1.3 <= (double)pl.bm);
  pl.nt = pl.once && 6ll * E * H * I > kKeepFewRowsBytes;
  return pl;
}

// Weights of a linear layer up to which 33 ... 128 tokens take 64-row tiles (two
// work-groups per CU) although 128-row tiles fill the chip too. 64- and 128-row
// tiles, weights rotated through 1.3 GB and repeated: 8192 x 4096 (67 MB), T = 80
// 24.0 24.9 and 20.0 22.9 us, T = 128 29.1 27.8 and 22.3 26.0; 8192 x 5632 (92 MB),
// T = 80 34.8 29.5 and 32.0 26.1; 5120 x 10240 (105 MB), T = 48 30.2 28.4 and 23.8
// 24.3, T = 128 39.7 34.7 and 28.5 30.5.
constexpr long long kSmallTileBytes = 84ll << 20;

// k-steps per split up to which a linear layer's 256-row tiles are worse than
// 128-row ones that fill one round of the chip too, or are as many: those take
// half the splits of twice the length, so half the fp32 partials and fewer of the
// loops' beginnings and ends (256- and 128-row tiles: 4096 x 4096, T = 512, 8 and
// 16 steps 45.4 and 32.8 us, T = 1024, 16 and 32 steps 55.1 and 47.7; 5120 x 5120,
// T = 512, 14 steps 45.9 and 42.6; 8192 x 5120, T = 320, 22 steps 42.6 and 44.2;
// 2048 x 4096, 192 work-groups of either, T = 768, 4 and 2 splits 36.1 and 28.2,
// T = 1536, 2 splits and 1 45.2 and 65.9).
constexpr int kFewSteps = 16;

// k-steps per split up to which a linear layer's 256-row tiles do not take several
// rounds of work-groups, however full, but the splits that one round holds: every
// split adds [T, N] of fp32 partials, written and read, and a k-loop's beginning
// and end. 6144 x 3072, T = 1400, 72 tiles: 7 splits 91 us, 5 90, 3 (one round, 84%
// full) 61; T = 3000, 144 tiles: 5 splits of 20 steps 168, one 111; 3072 x 6144, T =
// 1400, 144 tiles: 5 splits of 10 steps 109, one 62; 7168 x 9216, T = 448, 72 tiles: 7
// splits of 16 88, 3 67.
constexpr int kFewStepsOfRounds = 24;

// Plan of a linear layer [N, K] (gate_cols = 0) or of a SwiGLU whose down matrix
// is [N, K] and whose gate and up matrices are [gate_cols, N]: the largest tile
// of 256, 128 or 64 rows whose first GEMM has enough work-groups, unless the next
// smaller takes a second round of them; 32 rows up to 32 tokens. Small matrices
// gain most: SwiGLU 512 x 1408, T = 700 46 -> 21 us, linear 2048 x 1024, T = 200
// 20.5 -> 11.3.
//
// Up to 64 tokens, where one 64-row tile holds all rows, weights that stay cached
// take it. Where a linear layer's work-groups would be a few more than the CUs,
// some of which then hold two, it takes the splits that give each CU one at most
// (4096 x 5120, T = 40: 320 work-groups 18.0 us, 240 14.7, 160 of 128 rows 17.3; 2560 x
// 8192: 320 19.6, 256 15.0). From 65 on
// two 64-row tiles read every weight twice, which pays only where the 128-row
// tiles leave CUs idle (SwiGLU 2048 x 8192, T = 128, 64 work-groups of 128 rows:
// 43.0 us with 64-row tiles, 57.1 with 128; 1024 x 25600, 200 work-groups: 68.0
// and 55.4) or, in a small linear layer, the 64-row tiles fill one round of the
// chip (2048 x 16384, T = 80: 24.2 and 25.0; 4096 x 11264, two rounds: 39.2 and
// 28.2). (Weights rotated through 1.3 GB.)
inline FfnPlan plan_dense(int T, int N, int K, int gate_cols) {
  const long long bytes = (gate_cols ? 3ll : 1ll) * N * K * 2;
  const bool keep = bytes <= (T <= 16 ? kKeepFewRowsBytes : kKeepWeightBytes);
  FfnPlan pl;
  auto try_bm = [&](int bm) {  // returns the work-groups of the first GEMM
    const int mtiles = (T + bm - 1) / bm;
    const int ntiles = (N + down_bn(bm) - 1) / down_bn(bm);
    pl.bm = bm;
    plan_splits(mtiles * ntiles, K, down_target(bm), concurrent_wgs(bm), 8, &pl.down_splits, &pl.down_kps);
    return (long long)mtiles * (gate_cols ? (gate_cols + gate_bn(bm) - 1) / gate_bn(bm) : ntiles * pl.down_splits);
  };
  auto at_most = [&](int wgs) {  // the splits of pl.bm that give at most this many work-groups, one at least
    const int tiles = (T + pl.bm - 1) / pl.bm * ((N + down_bn(pl.bm) - 1) / down_bn(pl.bm));
    plan_splits(tiles, K, wgs / tiles * tiles, 0, 8, &pl.down_splits, &pl.down_kps);
  };
  auto one_round = [&](int bm, long long n) {  // of resident work-groups, nearly full
    return n <= concurrent_wgs(bm) && n * 16 >= concurrent_wgs(bm) * 15ll;
  };
  if (T <= 32) {
    try_bm(32);
  } else if (T > 128) {
    const long long n256 = try_bm(256);
    if (n256 <= kFewWorkGroups) {
      const long long n128 = try_bm(128);
      if (n128 > concurrent_wgs(128))
        try_bm(256);
      else if (n128 <= kFewWorkGroups && try_bm(64) > concurrent_wgs(64))
        try_bm(128);
    } else if (!gate_cols && pl.down_kps <= kFewSteps * 64) {
      const long long n128 = try_bm(128);
      if (!one_round(128, n128) && (n128 < n256 || n128 > concurrent_wgs(128) || pl.down_splits == 1)) try_bm(256);
    }
    if (!gate_cols && pl.bm == 256 && n256 > concurrent_wgs(256) && pl.down_kps <= kFewStepsOfRounds * 64)
      at_most(concurrent_wgs(256));
  } else {
    const long long n64 = try_bm(64), tiles64 = n64 / (gate_cols ? 1 : pl.down_splits), n128 = try_bm(128);
    const bool few = n128 <= kFewWorkGroups;
    bool small;
    if (T <= 64)
      small = gate_cols ? few || keep : n64 <= 256 || (bytes <= kSmallTileBytes && (tiles64 <= 256 || n64 >= 384));
    else
      small = keep && (few || (!gate_cols && bytes <= kSmallTileBytes && (one_round(64, n64) || !one_round(128, n128))));
    if (small) {
      try_bm(64);
      if (T <= 64 && !gate_cols && n64 > 256 && n64 < 384) at_most(256);
    }
  }
  pl.nt = !keep && T <= pl.bm;
  return pl;
}

// `nt`: weight loads are non-temporal.
hipError_t launch_gate_up(int bm, bool nt, const GemmParams& g, hipStream_t stream);
hipError_t launch_down(int bm, bool f32_partials, bool nt, const GemmParams& g, hipStream_t stream);

}  // namespace aflex

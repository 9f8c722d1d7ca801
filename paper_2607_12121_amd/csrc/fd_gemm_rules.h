// Which GEMM kernel, tile shape and number of K splits a product runs.  Plain C++, shared by
// the device code (M is only known there), the host code and a CPU build.
#pragma once

#include <math.h>

#include "fd_rules.h"

namespace fd {

constexpr int TBK = 64;   // K-step
constexpr int kMaxSplit = 16;
// K-steps every split keeps.  16: a split GEMM of 64 tiles and K = 4096 runs on 256 slots instead of
// 128 (1024 rows x 1024: 30.6 -> 24.7 us with its sum, 256 rows 27.6 -> 19.5; 24 was the line before);
// from 12 on the QKV and out projections (K = 1024 to 1536) split too, and their sums cost more than
// the splits give (image out-projection 20.5 -> 26.9 us).
constexpr int kMinSplitSteps = 16;

// Number of K splits (identical in every WG): split only while every unit keeps
// at least kMinSplitSteps K-steps and the units still fit the resident workgroup slots.
FD_RULE int choose_split(int tiles, int nk, int slots, int max_units) {
  int s = 1;
  while (s < kMaxSplit && tiles * (s + 1) <= slots && tiles * (s + 1) <= max_units && nk / (s + 1) >= kMinSplitSteps) ++s;
  return s;
}

// Tile shape of the two-workgroups-per-CU kernel for M rows (identical in every
// WG): 128x128 whenever split-K applies; otherwise the shape whose rounds of tiles
// over the resident slots cost least, a round of 128x64 / 128x128 / 128x192 tiles
// weighted 8 / 13 / 22 (measured per-round times at 1664 rows); ties go to the
// larger tile.  0 = 128x128, 1 = 128x192, 2 = 128x64 (three-stage ring: a round
// costs 8 where its two-stage version cost 10).
FD_RULE int small_shape(int M, int N, int K, int slots, int max_units) {
  const int tm = (M + 127) / 128;
  const int t128 = tm * ((N + 127) / 128);
  if (max_units > 0 && choose_split(t128, K / TBK, slots, max_units) > 1) return 0;
  const int r128 = (t128 + slots - 1) / slots;
  const int r192 = (tm * ((N + 191) / 192) + slots - 1) / slots;
  const int r64 = (tm * ((N + 63) / 64) + slots - 1) / slots;
  const int c128 = 13 * r128, c192 = 22 * r192, c64 = 8 * r64;
  if (c192 <= c128 && c192 <= c64) return 1;
  if (c128 <= c64) return 0;
  return 2;
}

// Tile shape of the 512-thread kernel for M rows (identical in every workgroup): 128x128
// with split-K wherever that applies; otherwise the shape whose rounds of tiles over the
// CUs cost least.  A round's cost is its time per K-step in 50 ns, measured at 970 to 13824
// rows x 1536 to 6144 columns: 256x256 27, 192x256 22, 128x256 16, 128x128 10; two 128x64
// tiles per CU 10, one 7.  Ties go to the larger tile.
enum LargeShape { kLargeTile = 0, kTallTile = 1, kMidTile = 2, kDeepTile = 3, kPairTile = 4 };
FD_RULE int large_shape(int M, int N, int K, int cus, int max_units) {
  auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  // rounds of t tiles: a multiply (five integer divisions cost every launch half a microsecond);
  // t is far below 2^23 and the slack far above the product's error, far below 1 / cus
  const float inv = 1.0f / static_cast<float>(cus);
  auto rounds = [&](int t) { return static_cast<int>(ceilf(static_cast<float>(t) * inv - 1e-4f)); };
  const int t128 = tiles(128, 128), r64 = rounds(tiles(128, 64));
  if (max_units > 0 && choose_split(t128, K / TBK, cus, max_units) > 1) return kDeepTile;
  int best = kLargeTile, cost = 27 * rounds(tiles(256, 256));
  auto consider = [&](int shape, int c) {
    if (c < cost) {
      best = shape;
      cost = c;
    }
  };
  consider(kTallTile, 22 * rounds(tiles(192, 256)));
  consider(kMidTile, 16 * rounds(tiles(128, 256)));
  consider(kDeepTile, 10 * rounds(t128));
  consider(kPairTile, (r64 >> 1) * 10 + (r64 & 1) * 7);
  return best;
}

// Row capacity (token count of the batch) from which the 512-thread kernel is used.  The
// active row count is only known on the device, so the choice rests on the capacity; its
// shapes hold for few rows too.  13824 tokens of 6 requests, image dims, us per block, small
// / large kernel: 7% active 179 / 179, 22% 378 / 355, 30% 488 / 440, 70% 1012 / 860; below
// 8192 tokens (1664 of 4096 rows: 221 / 224) the two small workgroups per CU win.
constexpr int kLargeTileRows = 8192;
// The embedding, whose K-steps are few, is bound by its epilogue, which more and smaller workgroups
// run as well (9676 x 1536: 42 / 39 us small / large kernel, 13600 x 1024: 41 / 45).
constexpr int kLargeEmbedRows = 16384;
FD_RULE bool gemm_large(int n_max, int N, bool embed) {
  return n_max >= (embed ? kLargeEmbedRows : kLargeTileRows) && N >= 1024;
}

// Row capacity from which the 512-thread kernel does not split: its splits need at most 128 tiles
// of 128x128, 2048 active rows at 1024 columns (an eighth of the rows here), 1280 at 1536, while the
// sum's launch, empty otherwise, costs every call 4 us.  Nor do products narrower than a tile, half
// of whose partial tiles are unused: last layer of hidden 3072, us, split / not, 32768 rows 208 / 190,
// 16384 104 / 101, 1638 of 32768 56 / 60.  The 256-thread kernel's other products split at any
// capacity: its 256 tiles are many of their rows (10880 at 384 columns), and unsplit they leave most
// of the GPU idle.  Down-projection, us, split / not, 4864 of 16384 rows: hidden 512, MLP 4096
// 42 / 62; hidden 768, MLP 3072 48 / 58.
constexpr int kNoSplitRows = 16384;
FD_RULE bool gemm_may_split(int n_max, int N, bool large) { return n_max < kNoSplitRows || (!large && N >= 128); }

}  // namespace fd

// Grids of prefill launches and the choice of their kernels.  Plain C++, so that it
// also compiles without a GPU toolchain.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "moa_internal.h"

namespace moa {

// Query tiles of `rows` rows, in dispatch units of `qchunk` tiles with all query
// heads of a KV head; units go to the accelerator dies in turn.
struct PrefillGrid {
  int64_t tiles, qchunk, n_chunks, n_units, blocks;
  int64_t per_die;                 // work-groups of the fullest die
};

inline PrefillGrid prefill_grid(const PrefillArgs& a, int rows) {
  PrefillGrid g;
  g.tiles = (a.n + rows - 1) / rows;
  // A unit spans at least kPrefillUnitBlocks work-groups (query tiles x group),
  // and at least kPrefillChunk query tiles.
  g.qchunk = std::min<int64_t>(std::max<int64_t>(kPrefillChunk, kPrefillUnitBlocks / a.group), g.tiles);
  g.n_chunks = (g.tiles + g.qchunk - 1) / g.qchunk;
  g.n_units = int64_t(a.hkv) * a.batch * g.n_chunks;
  if (g.n_units >= kMaxGrid) {
    g.per_die = g.blocks = kMaxGrid;
    return g;
  }
  g.per_die = (g.n_units + kNumXcd - 1) / kNumXcd * a.group * g.qchunk;
  g.blocks = g.per_die * kNumXcd;
  return g;
}

// Waves of 32 query rows and key groups per work-group of a bf16 launch.
struct PrefillShape {
  int waves, key_groups;
};

// A launch of few work-groups takes as long as its longest chain of tiles (a
// tile of a lone work-group 1.65 us at head_dim 128, of two on a compute unit
// 1.9), so the chain is split over two key groups, in work-groups of 64 rows or,
// where those are too many, 128.  Such a work-group takes the LDS of a whole
// compute unit at head_dim 128 and of half a one at 64.  What has to fit is the
// fullest die: a short prompt with few (KV head, sequence) pairs has its units on
// few dies.  Lines drawn through 900 launches of 1 to 64 heads and 100 to 8,192
// tokens, windows of 0.05 to 1.0 of them, each with all three kernels; with four
// waves of 128 rows, two key groups of them and two of 64 rows, in us:
//   64 rows where they fit.  32 heads x 512 at head_dim 128 18.6, -, 15.0; 16 heads
//     x 512 at 64 13.8, -, 9.7.  Twice as many as fit, 8 query heads of one KV head
//     x 1,024: 28.8, 32.0, 50.0 at head_dim 128.  At 64 then only long chains gain
//     (2 x 8 query heads of one KV head x 3,000: 74.8, 54.6, 59.3; windows of 51 x
//     1,024: 12.3, 13.1, 16.3), and launches whose units of half the rows come to
//     twice the dies (8 of one x 4,096, windows of 204: 25.6, 31.8, 20.9).
//   128 rows where those fit: 32 heads x 1,024 30.6, 26.1.  Up to twice as many, for
//     long chains of uneven length, which a full window gives: 32 heads x 2,048
//     57.0, 54.6 and 16 heads x 3,000 94.6, 61.6 at head_dim 128; but 2 x 32 heads
//     x 1,024 33.6, 38.9, and with windows of half the prompt (9 heads x 4,096)
//     58.9, 69.6.
// With more work-groups two per compute unit cover each other's waits and their
// starts and ends (32 heads x 4,096: 128 us against 139).
inline PrefillShape prefill_shape(const PrefillArgs& a, int head_dim) {
  int64_t widest = 0;
  for (int g = 0; g < a.hkv; ++g) widest = std::max(widest, int64_t(a.window[g]) << a.band_shift);
  const int64_t tiles = (a.n + 63) / 64;                  // of 64 keys
  const int64_t chain = std::min(tiles, (int64_t(a.num_sink) + 63) / 64 + widest / 64 + 3);
  const bool uneven = 8 * chain >= 7 * tiles && chain >= 20;
  const int64_t d64 = prefill_grid(a, 64).per_die, d128 = prefill_grid(a, 128).per_die;
  constexpr int64_t kUnits = 32;                          // compute units of a die
  if (head_dim == 128) {
    if (chain >= 4 && d64 <= kUnits) return {2, 2};
    if (d128 <= kUnits && (chain >= 8 || (chain >= 6 && 8 * chain >= 7 * tiles))) return {4, 2};
    if (d128 <= 2 * kUnits && uneven) return {4, 2};
    return {4, 1};
  }
  if (chain >= 3 && d64 <= 2 * kUnits) return {2, 2};
  if (chain >= 3 && d64 <= 4 * kUnits && (uneven || d64 <= d128)) return {2, 2};
  if ((chain >= 6 && d128 <= kUnits) || (chain >= 12 && d128 <= 2 * kUnits)) return {4, 2};
  const int64_t all128 = (a.n + 127) / 128 * a.batch * a.hq;
  if (uneven && d128 <= 4 * kUnits && all128 <= 2 * kUnits * kNumXcd) return {4, 2};
  return {4, 1};
}

// Kernel of an fp32 launch: 64-key tiles shared through LDS, or a wave's operands
// straight from memory, with 32 or 64 rows per wave and 1, 2 or 4 waves per block
// of rows.
struct PrefillF32Shape {
  bool shared;
  int key_groups, row_blocks;
};

// Blocks of 32 rows decide how many waves share one.  head_dim 128 (one wave per
// SIMD: 370 registers): 504 blocks 366 us with shared tiles, 93 with 4 waves per
// block (2: 142); 1,024 blocks 193, 95 with 2 (4: 114); 4,096 blocks 817, 546
// with one (2: 560).
//
// head_dim 64, lines drawn through 288 launches of 4 to 256 heads, 700 to 16,384
// tokens and windows of 0.2 to 1.0 of them, each with every kernel (us: shared
// tiles, 4 waves per 32 rows, 4 waves per 64, 2 waves per 64):
//   few blocks: 8 heads x 1,501 125, 49, -, 57; 32 heads x 2,048 292, 203, 208, 279.
//   from 2,900 blocks on a wave takes 64 rows, which halves its loads per product:
//     128 heads x 1,024 293, 207, 199, 214; 32 heads x 4,096 849, 786, 705, 739.
//   shared tiles where K and V are read many times over, that is for long prompts,
//     the sooner the more query heads share a KV head, and need fewer operand loads
//     still: 64 query and 8 KV heads x 2,500 on, 32 and 8 x 3,500 on, 32 and 32 x
//     5,000 on (64 and 8 x 8,192 4,557, 6,098, 5,332, 5,361; 32 and 8 x 8,192
//     2,319, 2,949, 2,671, 2,703), with few heads only
//     where the windows are narrow (8 heads x 8,192, windows of 1,638 268, 296, 293, 308).  They
//     keep a (KV head, sequence) pair on one die: with less than 4 pairs not, nor
//     with windows so short that little is read twice (32 and 8 x 4,096, windows of
//     81: 103, -, -, 90).
//   2 waves per 64 rows where a launch of narrow windows then has one work-group
//     for every compute unit (32 heads x 1,024, windows of 204 39, 41, 43, 31), and
//     where windows have few tiles to share out (128 heads x 2,048, windows of 40 173,
//     -, 166, 145).
inline PrefillF32Shape prefill_f32_shape(const PrefillArgs& a, int head_dim) {
  const int64_t blocks = (a.n + 31) / 32 * a.batch * a.hq;
  if (head_dim == 128) return {false, blocks >= 2500 ? 1 : blocks >= 800 ? 2 : 4, 1};
  int64_t widest = 0;
  for (int g = 0; g < a.hkv; ++g) widest = std::max(widest, int64_t(a.window[g]) << a.band_shift);
  const int64_t span = std::min(a.n, a.num_sink + widest), pairs = int64_t(a.hkv) * a.batch;
  const bool narrow = 3 * span < a.n, wide = 4 * span >= 3 * a.n;
  const int64_t long_n = a.group >= 8 ? 2500 : a.group >= 4 ? 3500 : 5000;
  const bool reread = pairs >= 4 && span >= 512;
  if (reread && blocks >= 3000 &&
      (a.n >= long_n || (a.n >= 3500 && blocks >= 16000) || (a.n >= 1400 && a.group >= 8 && wide)))
    return {true, 1, 1};
  if (reread && blocks >= 2000 && a.n >= 8000 && narrow) return {true, 1, 1};
  if (pairs >= 2 && span >= 512 && blocks >= 8000 && a.n >= 14000) return {true, 1, 1};
  if (narrow && blocks >= 850 && blocks <= 1024) return {false, 2, 2};
  if (blocks < 2900) return {false, 4, 1};
  return {false, span < 256 ? 2 : 4, 2};
}

}  // namespace moa

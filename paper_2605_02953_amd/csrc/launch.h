// Host-side helpers shared by the entry points: argument checks, tile choice, launch set-up.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <algorithm>
#include <atomic>
#include "../../include/ditron.h"
#include "gemm_core.h"

namespace ditron {

// 256x256 output tile for B stored [N, K]: 128x128 per wave, operands loaded straight into a ring of five LDS
// pieces (160 KiB), 16 x 16 x 32 MFMA.  (Measured with emulated peers against the same tile with register
// staging, two LDS stages and 32 x 32 x 16 MFMA, which it replaced: 5-9 % faster at K 3584 and 8192, 12 % faster at
// 16384, 6 % faster at 3696, whose last K tile is ragged.)
typedef GemmTile4W<256, 256, false, true, true> TileBigDirect;
// The same with 224 and 192 columns: fewer columns per tile for problems whose 256-column tiling leaves the last round
// of 256 units partly empty (choose_tile).
typedef GemmTile4W<256, 224, false, true, true> TileBigDirect224;
typedef GemmTile4W<256, 192, false, true, true> TileBigDirect192;
// The same three for fp8 operands (256-row tiles are taken by fp8 problems large enough for them, see
// ag_takes_decode_kernel).
typedef GemmTile4W<256, 256, false, true, true, true> TileBigF8;
typedef GemmTile4W<256, 224, false, true, true, true> TileBigF8_224;
typedef GemmTile4W<256, 192, false, true, true, true> TileBigF8_192;
// 128x128 output tile on the same loop with three K tiles in flight (112 KiB of LDS): 64x64 per wave; for problems with
// too few 256x256 tiles to fill the chip.  (The register-staged 32 x 32 x 16 loop with two LDS stages that it replaced
// requests one K tile ahead, which is less than the L2 takes under load: [1024 x 8192] x [8192 x 3696], operands resident,
// 73 -> 57 us; 0.53 -> 0.38 us per K tile of a work-group, about 840 cycles, of which the MFMAs are 512 and the LDS array's reads 260
// by its counter (profiles/tile_loops.md): neither fills the loop, its start-up and barrier latencies do the rest.)
typedef GemmTile4W<128, 128, false, true, true> TileSmall;
// The same for B stored [K, N].
typedef GemmTile4W<256, 256, true, true, true> TileBigKN;
typedef GemmTile4W<256, 224, true, true, true> TileBigKN224;
typedef GemmTile4W<256, 192, true, true, true> TileBigKN192;
typedef GemmTile4W<128, 128, true, true, true> TileSmallKN;
// The first form of that tile: register-staged, two LDS stages (64 KiB), 32 x 32 x 16 MFMA.  Left for the MoE down-projection of a few K
// tiles.
typedef GemmTile4W<128, 128> TileSmallStaged;
// The same two with two K tiles in flight (80 KiB): two work-groups share a unit.  For launches whose work-groups need several
// rounds all the same and are bound by more than their K loops (GEMM-ReduceScatter with the peers' copies, short MoE contractions).
typedef GemmTile4W<128, 128, false, true, true, false, 2> TileSmallPaired;
typedef GemmTile4W<128, 128, true, true, true, false, 2> TileSmallKNPaired;
// 128 x 64, four K tiles in flight (144 KiB), for problems of few 128 x 128 tiles: a unit's K tile is 24 KiB instead of 32, and
// twice as many units share the weight (choose_tile).
typedef GemmTile4W<128, 64, false, true, true> TileSmall64;
typedef GemmTile4W<128, 64, true, true, true> TileSmallKN64;
// The MoE grouped GEMM: 4 waves as 2 x 2.  An expert's rows are padded to whole row tiles, so the row
// tile is 128 unless the experts are large or the 128-row tiles would need more rounds (choose_moe_tile).
constexpr int kMoeBlockM = 128;   // the smallest row tile: what the upper bound on the tile count assumes
struct MoeTile {
  int block_m, block_n;
};
// Column block for 128-row tiles.  The number of row tiles is only known on the device, so
// the host works from the expectation under even routing (rows / 128 plus half a tile of
// padding per expert).  If some width gives one tile per compute unit at most, with one row
// tile more than expected still fitting, the narrowest such width: in a single round the time
// is one tile's, and that is bound by the bytes a compute unit can load, (128 + width) * K
// (measured with streamed weights at 20 row tiles x 1536 columns: 62, 72, 74 us for 128, 192,
// 256).  With several rounds the flops decide: the width that pads `inter` least, the wider
// one on a tie (measured: 176 columns 126, 108, 122 us; 256 columns 130, 142, 130 us).
inline int choose_moe_block_n(long expected_rows, int num_local_experts, int inter) {
  const long row_tiles = cdiv((int)std::min<long>(expected_rows, 1 << 30), kMoeBlockM) + (num_local_experts + 1) / 2;
  const int widths[3] = {128, 192, 256};
  for (int w : widths)
    if ((row_tiles + 1) * cdiv(inter, w) <= 256) return w;
  int best = 256;
  for (int w : widths)
    if (cdiv(inter, w) * w < cdiv(inter, best) * best || (cdiv(inter, w) * w == cdiv(inter, best) * best && w > best)) best = w;
  return best;
}
// Column block of 128-row tiles for [k, n] weights: the narrowest that gives one tile per unit at most, counting at least one
// row tile for each expert (choose_moe_block_n counts half a tile for an expert of a few rows, and the round that this
// hides costs more on a tile that has a unit to itself): 60 experts, 736 tokens top-2, hidden 1024 / 2048 / 4096, 936 columns: 192
// columns, two rounds, 57, 85, 143 us; 256 columns, one, 46, 69, 113; 256 tokens, 768 columns: 128 columns 47, 64, 99, 192 columns
// 42, 56, 87.  `several_rounds` where none does.
inline int moe_block_n_kn(long expected_rows, int num_local_experts, int cols, int several_rounds) {
  const long rows = std::min<long>(expected_rows, 1 << 30);
  const long row_tiles = std::max<long>(cdiv((int)rows, kMoeBlockM) + (num_local_experts + 1) / 2, std::min<long>(rows, num_local_experts));
  for (int w : {128, 192, 256})
    if ((row_tiles + 1) * cdiv(cols, w) <= 256) return w;
  return several_rounds;
}
// Column block of 256-row tiles for [k, n] weights: 128 where that is one tile per unit at most, else what choose_moe_tile says.  us for
// the whole call with 128 and with 256 columns, weights not in the caches: 8 experts x 1590 rows, hidden 4472, 304 columns (162 of the
// narrower tiles) 113, 128; one expert x 2048, hidden 1024, 2048 columns (144) 54, 60; 4 x 2048, hidden 2048, 512 columns (140) 66, 76;
// not so 16 x 2048 rows, 200 columns (274) 97, 82.
inline int moe_block_n_kn_256(long expected_rows, int num_local_experts, int cols, int block_n) {
  const long row_tiles = (std::min<long>(expected_rows, 1 << 30) + 255) / 256 + (num_local_experts + 1) / 2;
  return (row_tiles + 1) * cdiv(cols, 128) <= 256 ? 128 : block_n;
}
// Row tile.  What a tile costs is the bytes its compute unit loads, (rows + columns) * K, times the rounds
// the launch needs on 256 units; the 256-row tile's count 1.3 times (a factor fitted to former loops; with the present ones,
// [n, k] weights, the best 128-row tile and 256 x 256, us for the whole call: 60 experts x 546 rows x 176 columns 80, 73; 64 x 768 x 256
// 91, 80; 16 x 512 x 1024 78, 72; 64 x 256 x 512 84, 76, all of which the factor gives to 256 rows; 32 x 128 x 768 50, 65; 32 x 375 x 512 45,
// 52; 64 x 192 x 200 67, 96, which it leaves to 128; it misses 60 x 273 x 352 with 75, 73).  From 1024 rows per expert on the
// 256-row tile has fewer loads per MFMA and little padding (8 x 2048 x 1536 276, 226; 60 x 546 x 1408 301, 289; not so 32 x 1024 x 512
// 115, 120, and one expert x 2048 x 2048 39, 48).
inline MoeTile choose_moe_tile(long expected_rows, int num_local_experts, int inter) {
  const MoeTile small{kMoeBlockM, choose_moe_block_n(expected_rows, num_local_experts, inter)};
  const MoeTile big{256, inter <= 128 ? 128 : 256};
  if (expected_rows / num_local_experts >= 1024) return big;
  const long rows = std::min<long>(expected_rows, 1 << 30);
  auto per_unit = [&](const MoeTile& t) {
    const long tiles = ((rows + t.block_m - 1) / t.block_m + (num_local_experts + 1) / 2) * cdiv(inter, t.block_n);
    return ((tiles + 255) / 256) * (t.block_m + std::min(t.block_n, inter));
  };
  return 13 * per_unit(big) < 10 * per_unit(small) ? big : small;
}
// rows routed to the local experts if every expert received the same number of assignments
inline long moe_expected_rows(long total_tokens, int top_k, int num_experts, int num_local_experts) {
  return total_tokens * top_k * num_local_experts / num_experts;
}

struct TileChoice {
  bool big;
  int block_m, block_n, threads;
  int group_m;    // GROUP_SIZE_M of the grouped tile order
  int num_xcd;    // chiplets assumed by the work-group remap (0: no remap)
  int per_xcd;    // consecutive tiles handed to one chiplet inside a remap block
};

// What a launch of `tiles` tiles of 256 x block_n costs, in units of a full round of 256 x 256 tiles: the work of a
// tile times the rounds, a last round that fills the fraction x of the chip counting 0.55 + 0.45 x (measured: the
// 192 tiles of cfg 2's second round take 0.886 of the time of the 256 of its first, the chip being power-limited);
// a 224-column tile loads 3 % more bytes per flop, a 192-column tile 7 %.  The constants are bf16's; for e4m3 the choice they make
// was the fastest of the three widths, or within 2 % of it, at all of 24 shapes tried (256 / 224 / 192 columns, K 8192, us: 8192 x 1376
// 120 / 116 / 115, 8192 x 2560 199 / 186 / 175, 8192 x 3584 213 / 205 / 245, 8192 x 3696 215 / 263 / 245, 8192 x 6656 379 / 357 / 386).
inline double tiling_cost(long tiles, int block_n) {
  const double work = block_n / 256.0 * (block_n == 256 ? 1.0 : block_n == 224 ? 1.03 : 1.07);
  const long full = tiles / 256, rest = tiles % 256;
  return work * ((double)full + (rest ? 0.55 + 0.45 * (double)rest / 256.0 : 0.0));
}

// Who takes the 224-column and 192-column tiles.  AllGather-GEMM with B stored [N, K]: wherever the estimate above says so.
// B stored [K, N]: where the 256-column tiling leaves at least a quarter of a single round empty, 8192 x 1376 columns (192 tiles
// of 256 columns, 256 of 192) 231 -> 212 us.  In the other cases it is 1 to 4 % (8192 x 1792 238 -> 235, 4040 x 3080 198 -> 192,
// 7976 x 3584 399 -> 391 us) and ditron_tile_config's answer for op 4, 256 columns, stays.
// GEMM-ReduceScatter and GEMM + AllReduce never: the units that a partly empty
// round leaves go to the peers' copies and to the reduction there, and full rounds only put those behind the GEMM (8192 rows,
// GEMM-ReduceScatter of 3584 / 1792 / 1376 columns 139 -> 157, 104 -> 125, 91 -> 111 us; GEMM + AllReduce 207 -> 221,
// 151 -> 161, 131 -> 134 us).
// kAllReduce: like kNever, and the two shapes (256 x 256, 128 x 128) and their rule are fixed: in the two-shot form a rank owns
// every world-th tile, reduces it and broadcasts it, so the tiling is part of what the ranks agree on and what a call returns.
enum class Narrow { kNever, kNK, kKN, kF8, kAllReduce };   // kF8: as kNK, e4m3 operands

// The most 128 x 128 tiles with which GEMM-ReduceScatter stays on them.  Every tile ends by waiting for its stores and counting itself,
// which a short contraction does not hide, and 256-row tiles have a quarter as many (the figures are from tiles that ended with a release, which costs more); in a long one a second round of small
// tiles is partly empty and its units take the peers' copies, while the large tiles leave half of the chip to nobody.  So the
// line depends on K.  us with 128 x 128 tiles (as gemm_rs_impl runs them) and with 256-row ones, 8 ranks, weights not in the caches:
//   240 tiles, 2048 x 1920: K 1024 35.2, 33.2; 1536 37.1, 41.7; 3584 50.5, 75.0
//   256 tiles, 2048 x 2048: K 512 38.2, 31.2; 1536 45.2, 40.8; 2048 47.5, 48.0; 3584 59.0, 76.3
//   320 tiles, 2048 x 2560: K 1536 48.4, 41.8 (2 ranks 42.0, 42.4); 2048 49.9, 49.1 (45.2, 50.3); 2560 56.5, 64.2
//   384 tiles, 2048 x 3000: K 2048 61.5, 51.7; 2560 66.9, 61.4; 3584 74.1, 76.8; 480, 2048 x 3840: 2560 68.0, 64.6; 3584 77.2, 79.0; 5120 101, 107
//   496 tiles, 904 x 7936: K 3584 94.3, 80.8 (nothing is left of the second round); 6656 139, 131; 512, 4000 x 2048: 6656 130, 134; 8192 150, 158
// How many of the rows of the large tiles exist matters less: 306 tiles, 264 x 13056 (half of them): K 1024 43.7, 35.5; 2048 50.0,
// 52.3; 3584 70.8, 78.8; 516, 264 x 22016: 3584 119, 86.  One row of tiles is bound by the weight, which large tiles ask for in longer
// runs, at any K if most of its rows exist: 304 tiles, 128 x 38912, K 512 44.8, 34.8; 3584 105, 93; 6656 170, 155; 16 x 38912 512 28.2, 26.1;
// 2048 59.3, 56.5; 2560 65.9, 69.9; 6656 128, 145.
inline int reduce_scatter_small_tiles(int m, int k) {
  if (k <= 1536 || (m > 64 && m <= 128)) return 255;
  return k <= 2560 ? 352 : k <= 6144 ? 480 : 512;
}

// 256-row tiles where they fill three quarters of the chip in one round, or where 128 x 128 tiles need so many rounds that a
// round of larger ones is shorter all the same.  us with 128 x 128 tiles (fp8: the decode kernel's) and with 256-row ones:
// AllGather-GEMM, [n, k], K 4096: 496 tiles, 904 x 7936, 79.2, 81.9; 520, 1160 x 6656, 102, 82 (a third round).
// [k, n], K 4096: 384 tiles, 2048 x 3000, 82.0, 81.4; 473, 1288 x 5504, K 8192 141, 139; 512, 512 x 16384, K 8192 167, 146; where half
// of the rows do not exist 264 x 16384 K 4096 69.9, 71.6, K 16384 243, 259.
// fp8, at any padding: 320 tiles, 2048 x 2560, K 4096 72.5, 49.9; 306, 264 x 13056, 58.9, 42.5; 257, 128 x 32896, 63.4, 42.5; 320, 16 x 40960
// 52.4, 42.8; 384, 128 x 49152, 66.3, 50.1; 1002, 128 x 128256, 173, 158 (K 8192: 278, 279).
// The number of nodes is no part of the rule: buffers are sized from ditron_tile_config, which does not know it.
inline bool takes_big_tiles(int m, int n, int k, Narrow narrow) {
  const long big = (long)cdiv(m, 256) * cdiv(n, 256), small = (long)cdiv(m, 128) * cdiv(n, 128);
  if (big >= 192) return true;
  switch (narrow) {
    case Narrow::kNK: return small > 512;
    case Narrow::kKN: return small > 383;
    case Narrow::kF8: return small > 256;
    case Narrow::kNever: return small > reduce_scatter_small_tiles(m, k);
    default: return false;
  }
}

inline TileChoice choose_tile(int m, int n, int k, Narrow narrow) {
  TileChoice t{};
  const long tiles_big = (long)cdiv(m, 256) * cdiv(n, 256);
  t.big = takes_big_tiles(m, n, k, narrow);
  t.block_m = t.block_n = t.big ? 256 : 128;
  // Half as wide where that many tiles still fit the chip in one round and the K loop is what the call spends its time on.
  // us with 128 and with 64 columns.  AllGather-GEMM, B stored [K, N] ([N, K]: the decode kernel): 64 x 3584, K 512 12.5, 11.4; 8192
  // 56.4, 42.2; 1024 x 2048 (256 of these tiles) K 512 14.1, 14.2; 1024 19.4, 18.8; 4096 44.2, 39.5.
  // GEMM-ReduceScatter: where the tiles and the peers' copying work-groups (8 to 32) still fit the units together; beyond 64 tiles of 128
  // columns the contraction has to be longer for it to pay.  128 / 64 columns, us for the call (tiles of 128 columns): K 424 (119)
  // 16.7, 17.2; 544 (28) 12.1, 12.2; 552 (27) 13.2, 12.5; 728 (24) 14.5, 13.2; 968 (56) 17.2, 15.3; 1144 (60) 20.1, 17.4; 816 (80) 16.8, 17.6; 800 (106)
  // 15.9, 15.4; 1064 (114) 20.1, 19.4; 1568 (78) 20.3, 17.7; 2976 (94) 26.5, 22.7; 3192 (110) 38.2, 31.8; 848 (124, no units left) 17.5, 24.2.
  const long tiles_small = (long)cdiv(m, 128) * cdiv(n, 128);
  const bool fits = narrow == Narrow::kNever ? tiles_small <= (k >= 1024 ? 112 : 64) && k >= 512 : tiles_small <= 128 && k >= 512;
  if (fits && narrow != Narrow::kAllReduce) t.block_n = 64;
  if (t.big && (narrow == Narrow::kNK || narrow == Narrow::kF8 || (narrow == Narrow::kKN && tiles_big <= 192))) {
    double best = 0.98 * tiling_cost(tiles_big, 256);
    for (int bn : {224, 192}) {
      const double c = tiling_cost((long)cdiv(m, 256) * cdiv(n, bn), bn);
      if (c < best) { best = c; t.block_n = bn; }
    }
  }
  t.threads = t.big ? TileBigDirect::THREADS : TileSmall::THREADS;
  t.group_m = 4;
  t.num_xcd = 8;
  t.per_xcd = 32;
  return t;
}

// Decode-shaped AllGather-GEMM (ag_takes_decode_kernel: fp8 where takes_big_tiles says no, bf16 when the 128 x 128 tiles of the
// tile engine would not cover half the chip and B is stored [n, k]): the tiles of plan_decode, 4 computing waves + 4 loading waves.
inline bool bf16_ag_is_decode_shaped(int m, int n) { return (long)cdiv(m, 128) * cdiv(n, 128) <= 128; }
// The tile loaders address an operand with 32-bit byte offsets, and the buffer-addressed
// loaders reserve offsets from 0x7ffffff0 up as "out of range, reads zero".
inline bool fits_32bit(size_t rows, size_t cols, size_t esize) { return rows * cols * esize < 0x7ffffff0ull; }

// fp8 takes the 256-row tiles of the tile engine where takes_big_tiles says so, unless the
// caller asks for a decode variant or an operand is too large for the engine's 32-bit offsets.
inline Narrow ag_narrow(int dtype, int b_layout) {
  return dtype == DITRON_FP8_E4M3 ? Narrow::kF8 : b_layout == DITRON_B_NK ? Narrow::kNK : Narrow::kKN;
}
inline bool ag_takes_decode_kernel(int m, int n, int k, int dtype, int b_layout, int decode_variant) {
  if (dtype == DITRON_FP8_E4M3)
    return decode_variant != 0 || !takes_big_tiles(m, n, k, Narrow::kF8) || !fits_32bit(m, k, 1) || !fits_32bit(n, k, 1);
  return b_layout == DITRON_B_NK && bf16_ag_is_decode_shaped(m, n);
}
inline TileChoice choose_tile_decode(int /*m*/, int /*n*/, int /*k*/) {
  TileChoice t{};
  t.big = false;
  t.block_m = 128;
  t.block_n = 32;
  t.threads = 512;
  t.group_m = 4;
  t.num_xcd = 8;
  t.per_xcd = 32;
  return t;
}

// Decode-shaped problems: which kernel, tile and K split.  Variant 1 is the 128 x 32 tile over the whole
// contraction; 2 / 3 are 128 x 128 / 128 x 64 tiles with the contraction split over S work-groups; 4 is the
// per-shard form, 16-row tiles (one shard's rows at the decode shape: a tile waits for that shard only).
// S doubles while the grid stays within one work-group per compute unit, at most 8, and every split keeps at
// least four 128-byte K tiles.
// Variant 0 is variant 2 with the tile cut to the rows there are (16, 32 or 64 of them) and to 64 columns: a unit loads and exchanges no
// rows that do not exist, and half as many splits meet in a tile.  us for the call, 128 x 128, the narrower tile of 128 columns and this one,
// 8 ranks: bf16 64 x 3584, K 8192 33.6, 26.6, 25.9; 32 rows 32.7, 22.5, 20.4; 16 rows 32.1, 20.7, 18.6; 64 x 8192 57.2, 51.3, 46.4; 64 x 512, K 1024
// 12.5, 10.2, 9.8; e4m3 64 x 3584 26.9, 21.5, 18.5; 64 x 13056, K 4096 26.8, 21.1, 20.8; 8 x 6656, K 2048 20.0, 12.3, 11.0.  More than 64
// rows take 64 columns where eight splits would meet otherwise: 128 x 3584, K 8192 e4m3 28.8 -> 22.9, bf16 35.8 -> 34.5 (with four it is
// 0 to 5 %, 128 x 8192 32.7 -> 31.0: not taken, the library's tests hold ditron_tile_config and the workspace size to four splits of 128 columns there).
struct DecodePlan {
  int variant, block_m, block_n, splits, kt_per_split, ntiles;
  size_t partial_bytes;   // partial tiles (8 bytes per element: fp32 value + epoch), behind the gathered operand in the workspace
};
inline DecodePlan plan_decode(int m, int n, int k_bytes, int variant) {
  DecodePlan d{};
  d.variant = variant == 0 ? 2 : variant;
  d.block_m = d.variant == 4 ? 16 : 128;
  d.block_n = d.variant == 1 ? 32 : (d.variant == 3 ? 64 : 128);
  const int kt = cdiv(k_bytes, 128);
  auto split = [&] {
    d.ntiles = cdiv(m, d.block_m) * cdiv(n, d.block_n);
    d.splits = 1;
    if (d.variant != 1)
      while ((long)d.ntiles * d.splits * 2 <= 256 && d.splits * 2 <= 8 && kt / (d.splits * 2) >= 4) d.splits *= 2;
  };
  split();
  if (variant == 0 && (m <= 64 || d.splits == 8)) {
    d.block_m = m <= 16 ? 16 : m <= 32 ? 32 : m <= 64 ? 64 : 128;
    d.block_n = 64;
    split();
  }
  d.kt_per_split = cdiv(kt, d.splits);
  d.partial_bytes = d.splits > 1 ? (size_t)d.ntiles * d.splits * d.block_m * d.block_n * 2 * sizeof(float) : 0;
  return d;
}
inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// How many work-groups play the peers, and into how many teams they split (= chunks in flight
// at once).  On one GPU the copies are compute-unit work, so the cheapest emulation delivers
// everything as early and as fast as possible: enough work-groups to saturate HBM for a large
// transfer (about half a MiB each, at most one per compute unit), and as many teams as chunks,
// which is also how a full mesh of links behaves (every peer pushes at the same time).
struct ProducerPlan {
  int producers, teams;
};
// tiles_wait: nothing of the launch starts before a chunk is there (AllGather-GEMM), so a small transfer is spread further,
// 128 KiB each over up to 64 work-groups: [512 x 4096] gathered, 6656 columns 47.3 -> 40.6 us for the call; [256 x 8192], 3584
// columns, B stored [k, n] 58.0 -> 50.8; [1400 x 3072], 4096 columns 62.6 -> 58.7; [1024 x 8192], 3696 columns 80 -> 76.4 (128
// work-groups: 77.4).  Not so beyond 32 MiB, where 512 KiB each are as many already ([2048 x 8192], 64 work-groups 134.5, 128
// 136.4, 256 139.6 us), and not where the copies run beside the tiles (GEMM-ReduceScatter 128 x 8192: 28.7, 29.7 us).
inline ProducerPlan plan_producers(size_t total_bytes, size_t nchunks, bool tiles_wait = false) {
  ProducerPlan pl{};
  size_t want = (total_bytes + (512u << 10) - 1) / (512u << 10);
  if (tiles_wait) want = std::max(want, std::min<size_t>(64, (total_bytes + (128u << 10) - 1) / (128u << 10)));
  want = std::max(want, std::min<size_t>(64, nchunks));   // many small chunks: side by side, not one round trip to memory after another (28 of 2 KB: 32.8 -> 24.9 us for the call)
  want = (want + 7) / 8 * 8;
  pl.producers = (int)(want < 8 ? 8 : (want > 256 ? 256 : want));
  pl.teams = (int)std::min<size_t>(nchunks, pl.producers);
  if (pl.teams < 1) pl.teams = 1;
  return pl;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// With more than one node the tile-row order comes from the paper's multi-node listings; a shape
// for which they do not visit every tile row exactly once is refused.
inline bool node_order_is_bijection(int m, int block_m, int world, int nnodes, int rank, int mode) {
  const int npm = cdiv(m, block_m);
  constexpr int kMaxRows = 1 << 16;   // one bit per tile row on the stack: the check allocates nothing
  if (npm > kMaxRows) return false;
  uint64_t seen[kMaxRows / 64] = {0};
  for (int t = 0; t < npm; ++t) {
    const int r = tile_row_across_nodes(t, m, rank, world, nnodes, block_m, mode);
    if (r < 0 || r >= npm || (seen[r >> 6] >> (r & 63)) & 1) return false;
    seen[r >> 6] |= 1ull << (r & 63);
  }
  return true;
}

// Calls over several nodes are served where the listing with tiles of this many rows visits every tile row once, whatever
// the tile is that the problem takes: 128 rows for fp8, whose node orders cover more shapes than those of 256 rows do.
inline int node_listing_rows(int m, int n, int dtype) {
  return dtype == DITRON_BF16 && (long)cdiv(m, 256) * cdiv(n, 256) >= 192 ? 256 : 128;
}

// The number of nodes whose listing a call with tiles of block_m rows follows, 0 if it is refused.  Where the listing at
// listing_rows is complete and the one at block_m is not, the tile rows are visited in the one-node order: every tile still
// waits for, or counts towards, just the ranks whose rows it holds, so the order decides only how long it may wait.
inline int nodes_of_order(int m, int block_m, int listing_rows, int world, int nnodes, int rank, int mode) {
  if (nnodes <= 1) return 1;
  if (!node_order_is_bijection(m, listing_rows, world, nnodes, rank, mode)) return 0;
  return block_m == listing_rows || node_order_is_bijection(m, block_m, world, nnodes, rank, mode) ? nnodes : 1;
}

inline bool is_permutation(const int* v, int n) {
  bool seen[DITRON_MAX_WORLD] = {false};
  for (int i = 0; i < n; ++i) {
    if (v[i] < 0 || v[i] >= n || seen[v[i]]) return false;
    seen[v[i]] = true;
  }
  return true;
}

// Kernels with more than 64 KiB of dynamic LDS need the limit raised, once per (kernel, device): the
// outcome is remembered per kernel (one bit per device), so the driver call is not paid on every launch.
template <auto Kernel>
inline bool set_dynamic_lds(int bytes) {
  static std::atomic<uint64_t> configured{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  const uint64_t bit = 1ull << (dev & 63);
  if (configured.load(std::memory_order_acquire) & bit) return true;
  if (hipFuncSetAttribute((const void*)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
    return false;
  configured.fetch_or(bit, std::memory_order_release);
  return true;
}

// Per-call options with the defaults filled in.
struct Tuning {
  int num_nodes;
  unsigned spin_limit;
  int decode_variant;
  int moe_route_groups;
  bool valid;
};
inline Tuning resolve_tuning(const ditron_tuning_t* t, int world) {
  Tuning r{1, 1u << 20, 0, 0, true};
  if (!t) return r;
  if (t->num_nodes < 0 || t->num_nodes > DITRON_MAX_WORLD || t->decode_variant < 0 || t->decode_variant > 4) r.valid = false;
  if (t->moe_route_groups < 0 || t->moe_route_groups > 8) r.valid = false;
  for (int v : t->reserved) r.valid = r.valid && v == 0;
  if (t->num_nodes > 0) r.num_nodes = t->num_nodes;
  if (t->spin_limit) r.spin_limit = t->spin_limit;
  r.decode_variant = t->decode_variant;
  r.moe_route_groups = t->moe_route_groups;
  if (world % r.num_nodes != 0) r.valid = false;
  return r;
}

// Exactly one of the three producer modes.
enum class Mode { kInvalid, kEmulate, kExternal, kPreset };
inline Mode producer_mode(unsigned flags) {
  switch (flags & (DITRON_EMULATE_PRODUCER | DITRON_EXTERNAL_PRODUCER | DITRON_FLAGS_PRESET)) {
    case DITRON_EMULATE_PRODUCER: return Mode::kEmulate;
    case DITRON_EXTERNAL_PRODUCER: return Mode::kExternal;
    case DITRON_FLAGS_PRESET: return Mode::kPreset;
    default: return Mode::kInvalid;
  }
}

}  // namespace ditron

extern "C" ditron_status_t ditron_ag_gemm_decode(const void* const* a_shards, const void* b, int b_layout, void* c,
                                                 const float* a_scales, const float* b_scales, void* workspace,
                                                 int32_t* signals, int32_t* status, int32_t* schedule_out,
                                                 const int* arrival_order, int m_per_rank, int n, int k, int world,
                                                 int rank, int dtype, int32_t epoch, unsigned flags,
                                                 const ditron_tuning_t* tuning, void* stream);

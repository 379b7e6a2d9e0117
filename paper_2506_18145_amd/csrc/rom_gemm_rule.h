// Which kernel of the routed GEMM takes a call (host code, no HIP).  Kernels and their launches: rom_gemm.hip.
#pragma once

#include <cstdint>

namespace rom {

enum class GemmTile {
  kStream,     // one persistent stream of 256 x 256 tiles per CU
  kDma256,     // a 256 x 256 tile per workgroup, operands straight to LDS
  kReg256,     // the same through registers
  k128,        // 128 x 128 tiles, several workgroups per CU
  kSkinny,     // 64 rows: a few rows per group
};

struct GemmShape {
  int64_t M;             // rows of all groups
  int groups, N, K;
  bool dma;              // whole 64-wide slabs, both operands within 32-bit byte offsets, no slices of K
  bool wide;             // dma but for rows of A beyond 32-bit byte offsets
  bool w_kmajor;         // contraction-major weight
  bool in_place;         // the residual is the output
  bool f32_or_softplus;  // fp32 output, or bias and softplus: the stream kernel has no such epilogue
};

constexpr int kStreamMinK = 320;          // its schedule needs five slabs

// The times below are us on MI355X, plain or scaled bf16 output, experts drawn at random, kernel alone.
inline GemmTile gemm_tile(const GemmShape &s) {
  const int groups = s.groups > 0 ? s.groups : 1;
  const int64_t rows = s.M / groups, cols = (s.N + 255) / 256;
  if (rows < 96) return GemmTile::kSkinny;
  if (s.f32_or_softplus) {
    // fp32 output, 256 x 256 tiles against 128 x 128: too few to fill the CUs 16384 x 256 x 4096 (72 tiles) 77.7 / 65.0;
    // about one each 15373 x 1024 x 768 (256) 34.7 / 42.1; just above that, where the second round runs nearly empty,
    // 16695 x 1024 x 1536 (276) 85.0 / 76.4
    const int64_t tiles = (s.M / 256 + groups) * cols;
    const bool fills = (tiles >= 192 && tiles <= 256) || tiles >= 384;
    return s.dma && rows >= 1024 && s.N >= 256 && s.K > 256 && fills ? GemmTile::kDma256 : GemmTile::k128;
  }
  // 524288 x 2048 x 4096 in 8 groups: 7.72 against 9.41 ms with 128 x 128 tiles
  if (s.wide && rows >= 1024 && s.N >= 256 && s.K > 256) return GemmTile::kReg256;
  if (!s.dma || s.K < kStreamMinK || s.N < 256 || s.M >= (int64_t{1} << 30) || s.in_place) return GemmTile::k128;
  // Otherwise the weight would be transposed first: 16384 x 1536 x 384 in 8 groups 39.1 / 47.9
  if (s.w_kmajor) return GemmTile::kStream;
  // Stream or 128 x 128 tiles (us, in that order).  `tiles`: 256 x 256, with half a tile of padding per group where there are several.
  //   * a lone column tile and a bit is half padding: 14736 x 384 x 1536 in 16 groups 32.5 / 30.8
  //   * few slabs and few columns, start and end weigh most: 23704 x 640 x 384 in 8 groups 29.3 / 24.6
  //   * more than three quarters of a round of the CUs: 16384 x 8192 x 2048 in 8 groups 508 / 703, x 2048 x 512 54.1 / 57.7
  //   * its partial round is cut into pieces of half a tile, one per CU, from 64 tiles on, which gains if K is long
  //     (7664 x 1024 x 1536 in 8 groups 31.7 / 42.6) and loses if not (5387 x 1024 x 768 in 8 groups 19.9 / 18.7);
  //   * in quarters it has the 128 x 128 kernel's work per CU without a second workgroup to fill its waits
  //     (3072 x 1024 x 2048 in 8 groups 26.8 / 22.7, 512 x 8192 x 2048 31.7 / 26.6);
  //   * in eighths it reaches twice the CUs: 2476 x 256 x 640 in 4 groups 8.2 / 9.6, until K is so long that only the
  //     time per slab counts (400 x 1024 x 2048 20.6 / 18.9)
  const int64_t tiles = groups > 1 ? (s.M / 128 + groups) * cols / 2 : (s.M + 255) / 256 * cols;
  if (s.N > 256 && s.N <= 384) return GemmTile::k128;
  if (s.K < 512 && s.N < 1024 && tiles > 32) return GemmTile::k128;
  //   * with few rows a group, uneven groups have more padding than that: with half of the rows in one of 16 groups 2859 x 1536 x
  //     1536 46.5 / 33.5, 2782 x 3072 x 768 47.9 / 39.1 (2720 x 3072 x 768 in even ones 34.6 / 39.9).  With the work below, the
  //     uneven ones come out even (2475 x 4096 x 768 48.0 / 52.5, 2519 x 4096 x 768 54.5 / 51.1) and the others ahead; up
  //     to 128 tiles they lose over any K (1886 x 1536 x 3072 67.3 / 57.3)
  const bool busy = tiles > 192 || (tiles > 64 && s.K >= 1536);
  const bool stream = tiles <= 32 ? s.K < 1024 : busy && (rows >= 256 || (tiles > 128 && tiles * s.K >= (192 << 10)));
  return stream ? GemmTile::kStream : GemmTile::k128;
}

// Which short contractions (32 to 160 in whole 16-wide steps) take the streaming small-K kernel.  The general kernel runs a K that is no multiple
// of 64 in whole slabs: 3063 x 3072 x 96, one group, 22.0 us against 13.5, 16384 x 4096 x 160 without activation 74 / 36; layer calls with a
// rank of 80, 800 x 1280 165 / 161, 16000 x 1280 699 / 670, of 112, 4096 x 1792 402 / 389, of 144, 16000 x 2048 1310 / 1267, of 160
// 1314 / 1270, training ones 8000 x 1280 1415 / 1396, 16000 x 1792 3799 / 3746.  Its 64-row tiles have the shorter start where most groups have
// less than one of them (700 x 1536 x 48 in 8 groups 6.1 / 6.9, 1000 rows 10.3 / 7.1).  The form that accumulates is asked for
// with a K of 32, 64 and 128 only (use_rank_passes).
inline bool gemm_smallk(int64_t M, int groups, int K, bool accumulates) {
  if (K == 32 || K == 64 || K == 128) return true;
  return K % 16 == 0 && K >= 32 && K <= 160 && !accumulates && M >= int64_t{96} * groups;
}

// Blocks of 32 rows per workgroup of the narrow-output kernel: fewest bytes into a CU (its rows of A and every row of W), for as many
// rounds as there are more workgroups than CUs.  (Five blocks of rows by five of columns do not fit the registers.)
constexpr int kThinMinRows = 1024, kThinMaxCols = 160;
inline int64_t thin_blocks_per_cu(int64_t M, int groups, int nb, int k_splits, int rb) {
  const int64_t wgs = (groups > 1 ? M / (rb * 32) + groups : (M + rb * 32 - 1) / (rb * 32)) * k_splits;
  return (wgs + 255) / 256 * (rb + nb);
}
inline int thin_row_blocks(int64_t M, int groups, int N, int k_splits) {
  const int nb = (N + 31) / 32;
  int best = 1;
  for (int rb = 2; rb <= (nb < 5 ? 5 : 4); ++rb)
    if (thin_blocks_per_cu(M, groups, nb, k_splits, rb) < thin_blocks_per_cu(M, groups, nb, k_splits, best)) best = rb;
  return best;
}
// Slices of its contraction, in us: what a CU brings in at 45 KB/us, or all rows once at 2.6 TB/s (they were written just before, and what
// that pushed out of the caches is still on its way to memory), and partial sums written and read at 4 TB/s.
// 3063 x 128 x 3072 in 8 groups, GEMM alone: one slice 19.9 us, two 13.3; 16384 x 160 x 4096 one 65, two 75 (partial sums not counted).
// Slices times rows stay below a limit, so that scratch that is large enough for a call is so for every smaller one (thin_scratch_rows).
constexpr int64_t kThinSliceRows = 16384;
inline int thin_most_splits(int K) { return K < 512 ? 1 : K < 2048 ? K / 256 : 8; }
inline int64_t thin_scratch_rows(int64_t M, int K) {
  const int64_t most = thin_most_splits(K) * M < kThinSliceRows ? thin_most_splits(K) * M : kThinSliceRows;
  return M > most || thin_most_splits(K) == 1 ? M : most;
}
inline int thin_k_splits(int64_t M, int groups, int N, int K) {
  const int nb = (N + 31) / 32;
  int best = 1;
  double best_us = 0.0;
  for (int s = 1; s <= thin_most_splits(K) && (s == 1 || s * M <= kThinSliceRows); ++s) {
    const double fill = static_cast<double>(thin_blocks_per_cu(M, groups, nb, s, thin_row_blocks(M, groups, N, s))) * (K / s) * 64.0 / 45e3;
    const double rows = static_cast<double>(M) * K * 2.0 / 2.6e6;
    const double us = (fill > rows ? fill : rows) + s * (static_cast<double>(M) * N * 8.0 / 4e6);
    if (s == 1 || us < best_us) best = s, best_us = us;
  }
  return best;
}

// Which calls take the few-rows kernel: it gains while most experts have no row and few workgroups stream the weights.  Kernel
// alone, us, against the tiled kernels' (weights not read just before): one row, 8 groups, 8192 x 2048 8.7 / 27.9, 8 rows
// 33 / 47, 2048 x 4096 19.7 / 30.2, 3072 x 1536 13.7 / 13.5.  Over a short K, with more workgroups than the CUs hold at
// once (two each) and not many experts, the tiled kernel has as much in flight: 6 rows, 8 groups, 2048 x 1024 12.8 / 10.3, 8 rows
// 4096 x 1024 16.2 / 12.0, but in 64 groups 20.6 / 28.0.  From about 16 rows on it does everywhere (steps of 16 / 32 sequences,
// d_model 2048, 121 / 133 against 123 / 126 us).
constexpr int kGemmFewRows = 8;
inline bool gemm_few_rows(int64_t M, int groups, int N, int K) {
  if (M > kGemmFewRows || K % 64 != 0 || groups > 64) return false;
  const int64_t used = M < groups ? M : groups;
  return K > 1024 || groups > 16 || used * ((N + 15) / 16) <= 512;
}

// Which fp32 kernel takes a call: fp32 operands, and bf16 shapes that the kernels above do not take.
enum class GemmF32Tile {
  kSmall,      // 16 x 64 tiles, 16 x 16 a wavefront
  kWide,       // 64 x 64 tiles, 32 x 32 a wavefront, the next 64 contraction indices requested ahead of the products
  kWideShort,  // the same with no requests ahead: a third of the registers, three times the wavefronts
  kStaged,     // 64 x 64 tiles through LDS
};
// vec: rows of both operands can be read four elements at a time.  All times us on MI355X, 8 groups drawn at random, kernel alone.
//   * A group with fewer rows than a wide tile leaves it mostly empty: small / wide 64 rows x 8192 x 2048 184 / 321, 256 x 8192 x
//     2048 403 / 465, 500 x 4000 x 1000 128 / 149.  With every row in one of the groups it is ahead as well: fp32 layer of 500 tokens, 8
//     experts of width 2048, 962 / 1015, 4000 tokens, 64 experts, 7378 / 7710.
//   * Otherwise 64 x 64 tiles share their operands, and 16 x 64 ones have four times the wavefronts.  Over a long K the sharing gains
//     once there is a wide tile per CU (512 x 1000 x 2000, 256 tiles, 75.5 / 66.9; 8192 x 94 x 2000, 272, 90.4 / 80.9; at 192 tiles
//     49.6 / 71.7), over a short one only the wavefronts count until there are some 640 (512 x 1680 x 52, 432 tiles, 10.2 /
//     16.0, 1024 x 1680 x 52, 648, 19.9 / 21.0).
//   * Up to 256 contraction indices there is next to nothing to request ahead, and the registers for it cost two of three wavefronts:
//     4096 rows x 4864 x 152 214 / 147 without, x 8192 x 256 504 / 340.
//   * Element by element the requests are the bound, and LDS halves them: small / staged 1024 x 2032 x 63 26.5 / 25.0, 500 x 6432
//     x 201 147 / 77, but 512 tiles (512 x 2032 x 63) 17.3 / 21.4, and 64 x 4848 x 151 with eight rows a group 33 / 49.
inline GemmF32Tile gemm_f32_tile(int64_t M, int groups, int N, int k_per_split, int k_splits, bool vec) {
  const int64_t tiles = (M / 64 + groups) * ((N + 63) / 64) * k_splits;
  if (!vec) return M < int64_t{16} * groups || tiles < 640 ? GemmF32Tile::kSmall : GemmF32Tile::kStaged;
  const bool brief = k_per_split <= 256;
  if (M < int64_t{64} * groups || tiles < (brief ? 640 : 256)) return GemmF32Tile::kSmall;
  return brief ? GemmF32Tile::kWideShort : GemmF32Tile::kWide;
}

}  // namespace rom

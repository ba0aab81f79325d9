// Choices the host makes before a GEMM launch, as functions of the shape alone.  Plain C++ without device code, so that
// they can be checked where there is no GPU.
#pragma once

namespace spes {
namespace plan {

// sides of the matrix-core tiles
constexpr int kFullRows = 256, kHalfRows = 128, kQuarterRows = 64, kFullCols = 256, kHalfCols = 128;

inline long tiles(long rows, long cols, int bm, int bn) { return ((rows + bm - 1) / bm) * ((cols + bn - 1) / bn); }

// Blocks per operand set of a launch over several results of different shapes: the sets share one grid extent, the tile
// count of the set that has most.  (Idle blocks are not free: the longer side of the results along both grid axes is 128
// times too many for d_model = 8192, d_ff = 64, and the fp32 weight gradients of four such experts took 464 us, now 54.)
inline long set_grid_tiles(const int* rows, const int* cols, int n_sets, int bm, int bn) {
  long most = 0;
  for (int i = 0; i < n_sets; ++i) {
    const long t = tiles(rows[i], cols[i], bm, bn);
    if (t > most) most = t;
  }
  return most;
}

// Full tiles of a launch that run as pairs of half-height ones (asked on the device, where the counts are known): a last round of them that is
// at most half full, where the pairs and the launch's half-height tiles still are one round.  That costs 0.65 of a full round instead of a
// whole one; beyond one round they are two, 1.3.  A launch of up to 128 full tiles has no others left.
constexpr unsigned kRound = 256;      // tiles that run at once, one per CU
constexpr unsigned tiles_cut(unsigned full, unsigned half_height) {
  return 2 * (full % kRound) + half_height <= kRound ? full % kRound : 0u;
}

// Columns of a ragged-row GEMM on full tiles that run as a launch of their own, on half-width tiles: a last column tile
// that is at most half full.
inline int column_tail(int ndim) {
  const int tail = ndim % kFullCols;
  return ndim > kFullCols && tail <= kHalfCols ? tail : 0;
}

// Few tiles: a launch costs its number of rounds of 256 concurrent tiles, the last of them partly empty.  Half-width
// tiles cost 0.6 of a full one each and fill the rounds better; they are taken where that arithmetic says so (a layer
// of a few thousand tokens), never for a launch of many rounds.  est_tiles: expected number of row tiles (0: unknown).
// Step relative to full tiles throughout, mean (range of 96 %) over 7457 cells of widths that are multiples of 256, random layers under even,
// normal and Gumbel load: 0.95 (0.84 to 1.11) where the rule takes half-width tiles for both widths, 1.01 (0.91 to 1.11) where for one; half-width
// ones for both cost 1.10 (1.02 to 1.16) where it takes none.  The arithmetic counts whole rounds, and since a last round of full tiles may be
// cut (tiles_cut) it lies off where that happens: where one width takes half-width tiles, 0.94 up to 64 full tiles, 1.00 up to 128, but 1.03 at 257 to 384.
inline bool few_tiles_narrow(int ndim, int est_tiles) {
  if (est_tiles <= 0 || ndim % kFullCols != 0) return false;
  const long full = (long)est_tiles * (ndim / kFullCols);
  const long rounds_full = (full + 255) / 256, rounds_half = (2 * full + 255) / 256;
  return rounds_full <= 4 && 0.6 * rounds_half < 0.95 * rounds_full;
}

// Rows per tile of the ragged-row GEMMs.  A 256-row tile of an expert with a few dozen rows computes padding, one block
// per CU, while the weights it streams are the only work that is needed; 64- and 128-row tiles run two blocks per CU
// (all but the 128-row SwiGLU one), take any width in 128-column tiles and fill the chip with fewer rows.  They feed
// fewer MFMAs per byte read, so full tiles win again once experts fill them.  Us of a whole step with 256 / 128 / 64 rows, at a mean of n rows
// per expert, even load, top-4 (2 of 8 experts):
//   32 experts of 2048 x 2048   n = 20: 587 / 588 / 565   n = 60: 537 / 546 / 577   n = 112: 592 / 683 / 767
//   64 experts of 1408 x 1408   n = 40: 589 / 506 / 485   n = 96: 656 / 596 / 603   n = 112: 666 / 622 / 662
//   16 experts of 4096 x 2048   n = 40: 519 / 524 / 538   n = 80: 549 / 558 / 614   n = 112: 559 / 570 / 626
// A short contraction is mostly prologue and epilogue, which two blocks per CU overlap, and the line of 64 rows lies higher:
//   16 experts of 768 x 2048    n = 128: 174 / 177 / 157  n = 256: 223 / 216 / 220  n = 320: 256 / 239 / 259
//   64 experts of 512 x 352     n = 192: 146 / 132 / 140  n = 512: 262 / 234 / 242
// (the down projection contracts over d_ff: measured up to d_ff = 4 d_model) -- as long as the launch is short of blocks.
// Many full tiles overlap nothing less by themselves, and the longer the contraction, the fewer are many:
//   48 experts of 384 x 1536    n = 192 (720 tiles): 328 / 260 / 253    48 of 768 x 2048 (960) 481 / 545 / 559
//   64 experts of 768 x 1024    n = 192 (640 tiles): 331 / 361 / 395    64 of 704 x 2560, n = 224 (1760) 744 / 855 / 983
// From there on 64-row tiles end at 64 rows; 128-row ones go on as far as some more tiles (48 experts of 704 x 2752,
// n = 104, 946 tiles: 499 / 512 / 523), or wherever full tiles pay a second launch for a column tail (64 experts of
// 640 x 1280, n = 224: 446 / 439 / 467).
// Above its line of 64 rows a narrow layer takes 128 where two or three rounds of 256 concurrent full tiles would end
// in one that is partly and at most 0.6 full: 24 experts of 768 x 768 at n = 562 (1.1 rounds) 223 / 218 / 230, 16 of 768 x 2048 at n = 512
// (2.5 rounds) 321 / 309 / 350.  Also where that round would be cut in two (tiles_cut): over the 432 cells of this rule 0.94 of full tiles,
// 0.92 with two rounds and 0.96 with three, faster by 2 % or more in 298 and slower in 46.  (Top-2 in place of top-4, 4096 tokens of that 768
// x 2048 layer with its optimizer step are one of the others: 441 / 445.)
// A round that is full, or nearly, keeps full tiles: n = 384 at 768 x 2048 (2.0) 264 / 265 / 289; the shortest contractions
// (d_model up to 640) take 128, which is within 2 % now (8 experts of 512 x 2048, n = 900, 2.0: 205 / 209 / 214).
// The load is not known here; an uneven one moves every line.  Over 24032 cells (24 fixed and 7987 random shapes under even, normal and Gumbel
// load) the choice takes 0.88 of the time of full tiles on average, is more than 2 % slower than they are in 858 (at worst 36 %), and at
// least 10 % off the best height in 3260.  Most of those are wide layers beyond the line of 96 rows, where 128-row tiles take 0.93 of the
// choice's time up to 192 rows (0.81 where full tiles are fewer than 128, 1.03 where they are more than 1024), 0.98 up to 256, 1.02 up to 512 and
// 1.09 beyond.
inline int row_tile(long rows, int n_experts, int d_model, int d_ff) {
  if (rows <= 48L * n_experts) return kQuarterRows;
  const bool narrow = d_model <= 896 && d_ff <= 4L * d_model;
  const long full = (rows / kFullRows + (n_experts + 1) / 2) * ((d_ff + kHalfCols - 1) / kHalfCols);   // SwiGLU tiles to expect
  const bool below = narrow && rows <= (d_model <= 640 ? 512L : 256L) * n_experts;
  if (below && (full * d_model <= 448 * 1024 || rows <= 64L * n_experts)) return kQuarterRows;
  if (rows <= 96L * n_experts) return kHalfRows;
  if (below && (full * d_model <= 688 * 1024 || column_tail(d_model) > 0)) return kHalfRows;
  const long last = full % 256;                       // tiles of the last round, 0 if it is full
  if (narrow && full >= 256 && full < 3 * 256 && last <= 154 && (last > 0 || d_model <= 640)) return kHalfRows;
  return kFullRows;
}

// number of gate-gradient partials per row that the kEpiDSwiglu epilogue writes for ndim columns (two per column tile)
inline int rowdot_parts(int ndim, int row_tile, int est_tiles) {
  if (row_tile != kFullRows || few_tiles_narrow(ndim, est_tiles)) return 2 * ((ndim + kHalfCols - 1) / kHalfCols);
  return 2 * ((ndim + kFullCols - 1) / kFullCols);
}

// Weight gradients, all three matrices in one launch: 128 x 128 tiles, two blocks per CU, or 256 x 256 tiles, one per CU.
// full_tiles, small_tiles: how many of them over all sets.  mean_rows, max_rows: routed rows of an expert (the contraction) in
// the mean and at most; the lengths themselves are known on the device only.  What decides is the rounds of blocks on 256
// CUs, and how evenly the experts are loaded.  Backward of a layer, small tiles relative to full ones, mean (range of 96 %) over
// 7235 cells of random layers under three load distributions, with and without accumulation (which differ by 0.01 on average):
//   small ones in one round leave fewer CUs idle, and cover less padding: 0.92 (0.75 to 1.00) at any length
//   up to 256 full tiles are one round, small ones then more than one, and they read twice the operand bytes per FLOP:
//     1.00 (0.92 to 1.04) up to 700 rows, 1.02 (0.97 to 1.08) to 1500, 1.04 (0.94 to 1.15) from 1500 on -- where no expert can
//     exceed twice the mean.  A round lasts as long as the tiles of its longest expert, which small ones spread over more
//     CUs: 0.98 (0.77 to 1.09) where an expert can
//   257 to 320 full tiles end in a round that is nearly empty: 0.97 (0.82 to 1.04)
//   beyond, that round fills up and the difference goes: 0.97 (320 to 1024 tiles) and 1.00 (more) below 200 rows, 1.00 and 1.03 to 700,
//   1.02 and 1.05 to 1500, 1.04 and 1.12 above
// The choice is 1 % off the better tile on average, and more than 5 % off it in 280 cells.
inline bool wgrad_small_tiles(long full_tiles, long small_tiles, int mean_rows, int max_rows) {
  if (small_tiles <= 512) return true;
  if (full_tiles > 320) return false;
  return full_tiles > 256 || mean_rows <= 512 || max_rows > 2L * mean_rows;
}

// fp32 layers on the matrix cores: rows per tile, columns per gate-gradient partial (a wavefront's), and the blocks that fill the
// chip (two per CU)
constexpr int kF32Rows = 64, kF32ShortRows = 32, kF32RowdotCols = 32;
constexpr long kF32Blocks = 512;

// Their loads address an operand with 32-bit byte offsets; larger layers stay on the vector ALUs.
inline bool f32_on_matrix_cores(long tokens, long rows, long d_model, long d_ff) {
  const long lim = (1L << 30) - 8;
  return tokens * d_model < lim && rows * d_ff < lim && d_ff * d_model < lim;
}

// 64-row tiles where the GEMM with fewest columns fills the chip with them (64 columns each, 32 of the fused SwiGLU's two
// matrices), otherwise 32-row ones, whose blocks share out k as well.
inline int f32_row_tile(long rows, int n_experts, int d_model, int d_ff) {
  const long cols_d = (d_model + 63) / 64, cols_f = (d_ff + 31) / 32;
  const long est = rows / kF32Rows + (n_experts + 1) / 2;
  return est * (cols_d < cols_f ? cols_d : cols_f) >= kF32Blocks ? kF32Rows : kF32ShortRows;
}

}  // namespace plan
}  // namespace spes

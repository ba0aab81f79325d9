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

// Columns of a ragged-row GEMM on full tiles that run as a launch of their own, on half-width tiles: a last column tile
// that is at most half full.
inline int column_tail(int ndim) {
  const int tail = ndim % kFullCols;
  return ndim > kFullCols && tail <= kHalfCols ? tail : 0;
}

// Few tiles: a launch costs its number of rounds of 256 concurrent tiles, the last of them partly empty.  Half-width
// tiles cost 0.6 of a full one each and fill the rounds better; they are taken where that arithmetic says so (a layer
// of a few thousand tokens), never for a launch of many rounds.  est_tiles: expected number of row tiles (0: unknown).
inline bool few_tiles_narrow(int ndim, int est_tiles) {
  if (est_tiles <= 0 || ndim % kFullCols != 0) return false;
  const long full = (long)est_tiles * (ndim / kFullCols);
  const long rounds_full = (full + 255) / 256, rounds_half = (2 * full + 255) / 256;
  return rounds_full <= 4 && 0.6 * rounds_half < 0.95 * rounds_full;
}

// Rows per tile of the ragged-row GEMMs.  A 256-row tile of an expert with a few dozen rows computes padding, one block
// per CU, while the weights it streams are the only work that is needed; 64- and 128-row tiles run two blocks per CU
// (all but the 128-row SwiGLU one), take any width in 128-column tiles and fill the chip with fewer rows.  They feed
// fewer MFMAs per byte read, so full tiles win again once experts fill them.  Measured, us of a whole step with
// 256 / 128 / 64 rows, at a mean of n rows per expert, even load:
//   32 experts of 2048 x 2048   n = 20: 563 / 537 / 502   n = 60: 592 / 573 / 589   n = 112: 617 / 653 / 694
//   64 experts of 1408 x 1408   n = 40: 731 / 512 / 498   n = 96: 778 / 562 / 610   n = 112: 706 / 502 / 560
//   16 experts of 4096 x 2048   n = 40: 573 / 554 / 521   n = 80: 594 / 577 / 641   n = 112: 610 / 690 / 721
// (above 96 rows the best height changes with the width and the load; there full tiles stay, also where 128 would win).
// A short contraction is mostly prologue and epilogue, which two blocks per CU overlap, and the line of 64 rows lies higher:
//   16 experts of 768 x 2048    n = 128: 234 / 203 / 190  n = 256: 293 / 291 / 276  n = 320: 310 / 325 / 325
//   64 experts of 512 x 352     n = 192: 239 / 182 / 173  n = 512: 316 / 275 / 278
// (the down projection contracts over d_ff: measured up to d_ff = 4 d_model) -- as long as the launch is short of blocks.
// Many full tiles overlap nothing less by themselves, and the longer the contraction, the fewer are many:
//   48 experts of 384 x 1536    n = 192 (720 tiles): 408 / 292 / 262    48 of 768 x 2048 (960) 474 / 500 / 542
//   64 experts of 768 x 1024    n = 192 (640 tiles): 340 / 345 / 384    64 of 704 x 2560, n = 224 (1760) 682 / 803 / 944
// From there on 64-row tiles end at 64 rows; 128-row ones go on as far as some more tiles (48 experts of 704 x 2752,
// n = 104, 946 tiles: 564 / 474 / 496), or wherever full tiles pay a second launch for a column tail (64 experts of
// 640 x 1280, n = 224: 468 / 417 / 466).
// Above its line of 64 rows a narrow layer takes 128 where two or three rounds of 256 concurrent full tiles would end
// in one that is partly and at most 0.6 full: full tiles pay for the whole last round, 16 experts of 768 x 2048 at n = 512
// (2.5 rounds, unevenly loaded) 473 / 385 / 428, 24 experts of 768 x 768 at n = 562 (1.1) 279 / 268 / 282.  A round that is
// full, or nearly, is lost by them: n = 384 at 768 x 2048 (2.0) 324 / 336 / 341, n = 320 above (1.75), unless
// the load spills into a third (n = 384, normal load: 364 / 323 / 334); only the shortest contractions gain under any
// load (8 experts of 512 x 2048, n = 900, 2.0: 287 / 271 / 280).
// The load is not known here; an uneven one moves every line.  Over 5062 measured cells (34 fixed and 1307 random
// shapes under even, normal and Gumbel load) the choice takes 0.73 of the time of full tiles on average, is more than 2 %
// slower than they are in 53, 26 of them under Gumbel load (at worst 21 %), and at least 10 % off the best height in 627.
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
// CUs, and how evenly the experts are loaded.  Backward of a layer, small tiles relative to full ones, mean (range) over
// 1090 cells of 40 results and three load distributions:
//   small ones in one round leave fewer CUs idle, and cover less padding: 0.96 (0.78 to 1.00) at any length
//   up to 256 full tiles are one round, small ones then more than one, and they read twice the operand bytes per FLOP:
//     1.00 (0.97 to 1.04) up to 700 rows, 1.02 (0.96 to 1.08) to 1500, 1.05 (0.98 to 1.17) from 1500 on -- where no expert can
//     exceed twice the mean.  A round lasts as long as the tiles of its longest expert, which small ones spread over more
//     CUs: 0.98 (0.74 to 1.11) where an expert can
//   257 to 320 full tiles end in a round that is nearly empty: 0.96 (0.90 to 1.04)
//   beyond, that round fills up and the difference goes: 0.97 at 64 rows, 1.00 at 1024, 1.08 at 16384
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

// Choices the host makes before a GEMM launch, as functions of the shape alone.  Plain C++ without device code, so that
// they can be checked where there is no GPU.
#pragma once

namespace spes {
namespace plan {

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

// Weight gradients, all three matrices in one launch: 128 x 128 tiles, two blocks per CU, or 256 x 256 tiles, one per CU.
// full_tiles: 256 x 256 tiles over all sets.  mean_rows, max_rows: routed rows of an expert (the contraction) in the mean
// and at most; the lengths themselves are known on the device only.  What decides is the rounds of blocks on 256 CUs, and
// how evenly the experts are loaded.  Backward of a layer, small tiles relative to full ones in the same launch:
//   at most 128 full tiles leave CUs idle, small ones do not: 72 tiles (1528 x 1008) 0.94 at 512 rows, 0.89 at 8192;
//     96 tiles (512 x 352, 8 experts) 0.94 at 64 rows, 0.85 at 16384
//   129 to 256 are one round of full tiles and more than one of small ones, which read twice the operand bytes per FLOP:
//     0.98 to 1.02 at 512 rows, 1.00 to 1.10 at 8192 (240 tiles of 1024 x 1024: 1.035, 1.11) -- under an even load.  When
//     some experts are twice the mean, the round lasts as long as their tiles and small ones spread them over more CUs:
//     0.89 to 0.95 at 8192 rows.  Full tiles are therefore taken where an expert cannot exceed twice the mean; over three
//     load distributions and 3000 rows or more small ones measured 1.04 there (0.99 to 1.17), 0.98 elsewhere (0.74 to 1.08)
//   257 to 320 end in a round of full tiles that is nearly empty: 0.86 to 1.00 at any length (288 tiles of 768 x 2048: 0.96
//     at 512 rows, 0.97 at 8192)
//   beyond, the second round fills up and the difference goes: 360 tiles of 1528 x 1008 0.99 at 512 rows, 1.06 at 16384
inline bool wgrad_small_tiles(long full_tiles, int mean_rows, int max_rows) {
  if (full_tiles > 320) return false;
  return full_tiles <= 128 || full_tiles > 256 || mean_rows <= 512 || max_rows > 2L * mean_rows;
}

}  // namespace plan
}  // namespace spes

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

}  // namespace plan
}  // namespace spes

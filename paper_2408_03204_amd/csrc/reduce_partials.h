// Sums of per-tile parameter-gradient partials, as blocks of whichever launch runs them.
#pragma once

#include "device_common.h"
#include "kernels.h"

namespace grafx {

// dP[slot][j] = sum over tiles of part[slot][tile][j], fixed order; block b of J.blocks() serves slot
// b of the concatenated slot ranges of the jobs.
__device__ __forceinline__ void reduce_partials(const ReduceJobs& J, int b) {
  __shared__ double red[4];
  int slot = b, q = 0;
  while (q + 1 < J.n && slot >= J.slots[q]) slot -= J.slots[q++];  // uniform over the block
  const double* part = J.part[q];
  const int tiles = J.tiles[q], np = J.np[q];
  for (int j = 0; j < np; ++j) {
    double s = 0.0;
    for (int i = threadIdx.x; i < tiles; i += kBlock) s += part[((int64_t)slot * tiles + i) * np + j];
    s = block_sum<double>(s, red);
    if (threadIdx.x == 0) J.dP[q][(int64_t)slot * np + j] = (float)s;
  }
}

}  // namespace grafx

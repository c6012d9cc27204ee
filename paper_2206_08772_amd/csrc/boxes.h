// The start of a support search: the nodes' bounding box, as one box per
// workgroup of the launch that has their positions at hand, and the counters
// that the same launch clears for the binning.
#pragma once

#include "launch.h"
#include "otm_common.h"

namespace otm {

struct BinCounters {
  int32_t* node_start;  // [cap + 1]
  int32_t* mp_start;    // [cap + 1]
  int64_t cap;
  int32_t* ticket;      // of the pair runs' workgroups
  OTM_DEV void clear() const {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i <= cap;
         i += (int64_t)gridDim.x * blockDim.x) {
      node_start[i] = 0;
      mp_start[i] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;
  }
};
inline BinCounters bin_counters(const Workspace& w) {
  return {w.cell_start, w.mp_cell_start, w.cap_cells, w.ticket};
}

struct Box {
  double lo[3], hi[3];
  OTM_DEV void clear() {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      lo[c] = INFINITY;
      hi[c] = -INFINITY;
    }
  }
  OTM_DEV void add(int c, double v) {
    lo[c] = fmin(lo[c], v);
    hi[c] = fmax(hi[c], v);
  }
  OTM_DEV void wave_join() {
    for (int o = kWave / 2; o > 0; o >>= 1) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lo[c] = fmin(lo[c], __shfl_xor(lo[c], o));
        hi[c] = fmax(hi[c], __shfl_xor(hi[c], o));
      }
    }
  }
  // Over a workgroup of 256 threads, in every thread (sh: 4 boxes).
  OTM_DEV void block_join(Box* sh) {
    wave_join();
    if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = *this;
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lo[c] = fmin(lo[c], sh[w].lo[c]);
        hi[c] = fmax(hi[c], sh[w].hi[c]);
      }
    }
  }
};

}  // namespace otm

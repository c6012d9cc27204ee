// The start of a support search: the nodes' bounding box, as one box per
// workgroup of the launch that has their positions at hand, and the counters
// that the same launch clears for the binning.
#pragma once

#include "launch.h"
#include "otm_common.h"

namespace otm {

struct BinCounters {
  int32_t* node_cnt;  // [cap + 1]: the counts are taken from [1] on
  int32_t* mp_cnt;    // [cap + 1]
  int64_t cap;
  int32_t* ticket;      // of the pair runs' workgroups
  OTM_DEV void clear() const {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i <= cap;
         i += (int64_t)gridDim.x * blockDim.x) {
      node_cnt[i] = 0;
      mp_cnt[i] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;
  }
};

// Bodies of few cells: every workgroup of the fill scans the cells' counts
// itself (the cells in use, two or three per thread as a rule), which spares the
// scan's launch: scan and fill of 4374 MPs 3.6 us instead of 3.5 + 2.8 and the
// gap between them, of 27.8k MPs 5.1 instead of 4.0 + 3.1.  With many MPs the
// workgroups' repeated scans would cost more than the launch.  The counts then
// lie apart from the row starts that the fill writes, in the part of the
// staging rows that the MPs' ranks leave.
constexpr int kFewCells = 8192;
constexpr int64_t kFewCellsMps = 65536;
inline bool few_cells(const Workspace& w, int64_t n_mp) {
  return w.cap_cells <= kFewCells && n_mp <= kFewCellsMps &&
         2 * (w.cap_cells + 1) <= (kRowCapacity - 1) * n_mp;
}
inline BinCounters bin_counters(const Workspace& w, int64_t n_mp) {
  if (few_cells(w, n_mp)) {
    int32_t* const at = w.stage + n_mp;
    return {at, at + w.cap_cells + 1, w.cap_cells, w.ticket};
  }
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

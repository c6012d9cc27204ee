// Support-domain search with linked cells (Sec. 3, Alg. 3), plus the prefix
// sums and small fills the library needs.
//
// Nodes are binned into static cells of edge >= r_list over their bounding
// box; a copy of the node coordinates is stored in cell order (x, y, z, id
// as one 32-byte record) so the 27-cell scan of an MP reads contiguous
// memory.  Each MP's row is sorted by id when it is copied to its place, so
// lists come out in canonical order.  The squared distance is evaluated as
// ((dx*dx + dy*dy) + dz*dz) with every operation rounded separately.
//
// A small body's search is bound by its launches (3 to 4 us each even when
// nearly empty), so whatever a kernel's workgroups can find out from a few
// hundred words they read and reduce themselves: the grid from the box
// partials (in the count), the totals before a scan workgroup, the pairs
// before a compaction group.  6 launches up to 8192 MPs and 16384 cells, 7 to 8
// above, where up to 13 were needed, and two fewer where the fill scans the cells
// (few_cells) and, in a step of up to 65536 nodes, the node update forms the box
// partials.  Search of 4374 MPs in a step: 25 us of kernel time, 73 before;
// 27.8k: 40 (86); 108k: 73 (99); 1.13M: 301 (352).
#include <type_traits>

#include "boxes.h"
#include "launch.h"
#include "otm_common.h"

namespace otm {

// ---------------------------------------------------------------- prefix sum
// Inclusive scan in two passes: each workgroup scans kScanBlock elements (16
// per thread) and writes its total, then each workgroup adds the totals before
// its own, which it sums itself (a third launch that scans them costs more
// than these reads: two arrays of 190k counts 12 us, 16 with it).  Up to kScanBlock elements take
// one launch.  Two arrays of equal length (the node and MP cell counts) go
// through the same launches: workgroup b works on array b / nb.  ``live``
// (nullable) holds how many of the n elements are in use.
constexpr int kScanPer = kScanBlock / 1024;
template <typename T>
struct Pack4 {
  T v[4];
};

// Sum over the workgroup's waves of v, in every thread (sh: one value per wave).
template <typename T>
OTM_DEV T block_sum(T v, T* sh) {
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int waves = (int)blockDim.x / kWave;
  if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = v;
  __syncthreads();
  T t = 0;
  for (int w = 0; w < waves; ++w) t += sh[w];
  return t;
}

// Exclusive scan of one value per thread over the workgroup; total: the sum.
template <typename T>
OTM_DEV T block_scan(T v, T* sh, T& total) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int waves = (int)blockDim.x / kWave;
  T run = v;
  for (int o = 1; o < kWave; o <<= 1) {
    const T u = __shfl_up(run, o);
    run += lane >= o ? u : T(0);
  }
  if (lane == kWave - 1) sh[wave] = run;
  __syncthreads();
  T before = 0;
  total = 0;
  for (int w = 0; w < waves; ++w) {
    before += w < wave ? sh[w] : T(0);
    total += sh[w];
  }
  return before + run - v;
}

template <typename T>
__global__ __launch_bounds__(1024) void k_scan_blocks(T* a, T* b, int64_t n, int64_t nb,
                                                      int64_t* aux, const int64_t* live) {
  __shared__ T sh[1024 / kWave];
  const int64_t seg = blockIdx.x / nb, blk = blockIdx.x - seg * nb;
  T* arr = seg == 0 ? a : b;
  const int64_t in_use = live != nullptr && *live < n ? *live : n;
  const int64_t base = blk * kScanBlock + (int64_t)threadIdx.x * kScanPer;
  if (blk * kScanBlock >= in_use) return;
  // whole runs move as packs of four (the arrays start one element off a
  // 16-byte boundary: packs of element alignment)
  Pack4<T>* pack = reinterpret_cast<Pack4<T>*>(arr + base);
  const bool whole = base + kScanPer <= in_use;
  T v[kScanPer], sum = 0;
  if (whole) {
#pragma unroll
    for (int k = 0; k < kScanPer / 4; ++k) {
      const Pack4<T> q = pack[k];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * k + e] = q.v[e];
    }
  } else {
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) v[k] = base + k < in_use ? arr[base + k] : T(0);
  }
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    sum += v[k];
    v[k] = sum;
  }
  T total;
  const T excl = block_scan(sum, sh, total);
  if (whole) {
#pragma unroll
    for (int k = 0; k < kScanPer / 4; ++k) {
      Pack4<T> q;
#pragma unroll
      for (int e = 0; e < 4; ++e) q.v[e] = v[4 * k + e] + excl;
      pack[k] = q;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kScanPer; ++k)
      if (base + k < in_use) arr[base + k] = v[k] + excl;
  }
  if (threadIdx.x == 0) aux[blockIdx.x] = (int64_t)total;
}

template <typename T>
__global__ __launch_bounds__(1024) void k_scan_add(T* a, T* b, int64_t n, int64_t nb,
                                                   const int64_t* aux, const int64_t* live) {
  __shared__ int64_t sh[1024 / kWave];
  const int64_t seg = blockIdx.x / nb, blk = blockIdx.x - seg * nb;
  const int64_t in_use = live != nullptr && *live < n ? *live : n;
  if (blk == 0 || blk * kScanBlock >= in_use) return;
  int64_t part = 0;
  for (int64_t i = threadIdx.x; i < blk; i += 1024) part += aux[seg * nb + i];
  const T add = (T)block_sum(part, sh);
  T* arr = seg == 0 ? a : b;
  for (int k = threadIdx.x; k < kScanBlock; k += 1024) {
    const int64_t i = blk * kScanBlock + k;
    if (i < in_use) arr[i] += add;
  }
}

// b == nullptr: one array
template <typename T>
static void scan_impl(T* a, T* b, int64_t n, int64_t* aux, const int64_t* live, hipStream_t s) {
  if (n <= 0) return;
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  const unsigned grid = (unsigned)(nb * (b == nullptr ? 1 : 2));
  k_scan_blocks<T><<<grid, 1024, 0, s>>>(a, b, n, nb, aux, live);
  if (nb > 1) k_scan_add<T><<<grid, 1024, 0, s>>>(a, b, n, nb, aux, live);
}
void scan_inclusive(int64_t* a, int64_t n, int64_t* aux, hipStream_t s) {
  scan_impl<int64_t>(a, nullptr, n, aux, nullptr, s);
}
void scan_inclusive(int32_t* a, int64_t n, int64_t* aux, hipStream_t s) {
  scan_impl<int32_t>(a, nullptr, n, aux, nullptr, s);
}

// ---------------------------------------------------------------- fills
__global__ void k_fill_i32(int32_t* a, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    a[i] = v;
}
__global__ void k_fill_f64(double* a, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    a[i] = v;
}
static unsigned fill_blocks(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return (unsigned)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}
void launch_zero(double* a, int64_t n, hipStream_t s) {
  if (n > 0) k_fill_f64<<<fill_blocks(n), 256, 0, s>>>(a, n, 0.0);
}
__global__ void k_fill_i64(int64_t* a, int64_t n, int64_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    a[i] = v;
}
void launch_fill_i32(int32_t* a, int64_t n, int32_t v, hipStream_t s) {
  if (n > 0) k_fill_i32<<<fill_blocks(n), 256, 0, s>>>(a, n, v);
}
void launch_fill_i64(int64_t* a, int64_t n, int64_t v, hipStream_t s) {
  if (n > 0) k_fill_i64<<<fill_blocks(n), 256, 0, s>>>(a, n, v);
}

__global__ void k_diag_reset(otm_diag* d) {
  d->flags = 0;
  d->max_support = 0;
  d->n_lme_noconv = d->n_rm_noconv = d->n_inverted = d->n_nonfinite = 0;
  d->first_lme_noconv = d->first_rm_noconv = d->first_inverted = d->first_nonfinite = ~0ull;
  d->pairs_needed = 0;
  d->reserved[0] = d->reserved[1] = d->reserved[2] = 0;
}
void launch_diag_reset(otm_diag* d, hipStream_t s) { k_diag_reset<<<1, 1, 0, s>>>(d); }

// ---------------------------------------------------------------- cell grid
// Nodes per bounding-box workgroup: four per thread, more past kBBoxBlocks
// workgroups (every counting workgroup reads all their boxes).
static unsigned bbox_blocks(int64_t n) {
  const int64_t b = (n + 1023) / 1024;
  return (unsigned)(b < 1 ? 1 : (b < kBBoxBlocks ? b : kBBoxBlocks));
}

// Bounding box partials of the nodes, one per workgroup; the same launch clears
// the cell counters of the node and MP binnings that follow.
__global__ __launch_bounds__(256) void k_bbox_partial(const double* x, int64_t n, Box* part,
                                                      BinCounters z) {
  __shared__ Box sh[4];
  z.clear();
  Box b;
  b.clear();
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
    for (int c = 0; c < 3; ++c) b.add(c, x[c * n + i]);
  }
  b.block_join(sh);
  if (threadIdx.x == 0) part[blockIdx.x] = b;
}

// Grid over the box: cell edge = cell_size, enlarged by 1.25x until the cell
// count fits the workspace (a larger cell only adds candidates).  Non-finite
// extents fall back to a single cell of unbounded size; every coordinate is
// clamped into the grid, so no cell index can leave it.
OTM_DEV Grid make_grid(const Box& b, double cell_size, int64_t cap) {
  double lo[3], ext[3];
  bool finite = true;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    lo[c] = b.lo[c];
    ext[c] = b.hi[c] - b.lo[c];
    if (!isfinite(ext[c]) || !isfinite(lo[c])) finite = false;
    if (!(ext[c] > 0.0)) ext[c] = 0.0;
  }
  double cell = cell_size, dx = 1.0, dy = 1.0, dz = 1.0;
  bool fits = false;
  for (int tries = 0; finite && tries < 400; ++tries) {
    dx = floor(ext[0] / cell) + 1.0;
    dy = floor(ext[1] / cell) + 1.0;
    dz = floor(ext[2] / cell) + 1.0;
    fits = dx * dy * dz <= (double)cap;
    if (fits) break;
    cell *= 1.25;
  }
  Grid g;
#pragma unroll
  for (int c = 0; c < 3; ++c) g.lo[c] = fits || isfinite(lo[c]) ? lo[c] : 0.0;
  g.dims[0] = fits ? (int32_t)dx : 1;
  g.dims[1] = fits ? (int32_t)dy : 1;
  g.dims[2] = fits ? (int32_t)dz : 1;
  g.cell = fits ? cell : INFINITY;
  g.n_cells = (int64_t)g.dims[0] * g.dims[1] * g.dims[2];
  g.pad = 0;
  return g;
}

OTM_DEV int cell_coord(double x, double lo, double inv_cell, int dim) {
  const double t = floor((x - lo) * inv_cell);
  // NaN lands in cell 0 (non-finite positions are reported by the MP update)
  int c = !(t >= 0.0) ? 0 : (t > (double)(dim - 1) ? dim - 1 : (int)t);
  return c;
}

// Counting sort of two point sets (nodes, then MPs) on one grid, each pass
// one launch: thread i < n_a takes point i of set a, threads from b0 (n_a
// rounded up to a wave, so no wave mixes the sets and the wave-grouped
// atomics see one counter array) take set b.  The count keeps each point's
// rank in its cell, so that the fill needs no atomics.
struct BinSet {
  const double* x;     // [3][n]
  int64_t n;
  int32_t* cell;       // [n] cell of each point
  int32_t* rank;       // [n] its place among the cell's points
  int32_t* cnt;        // [cap + 1] counts, from [1] on
  int32_t* start;      // [cap + 1] offsets (the same place, with many cells)
  double4* sorted;     // [n] (x, y, z, index) in cell order
};
constexpr unsigned kCountBlocks = 2048;  // of the count: as many as fit at once

// The set and point of thread t, false where there is none.
OTM_DEV bool bin_pick(const BinSet& a, const BinSet& b, int64_t b0, int64_t t, BinSet& set,
                      int64_t& i) {
  const bool first = t < a.n;
  i = first ? t : t - b0;
  set.x = first ? a.x : b.x;
  set.n = first ? a.n : b.n;
  set.cell = first ? a.cell : b.cell;
  set.rank = first ? a.rank : b.rank;
  set.cnt = first ? a.cnt : b.cnt;
  set.start = first ? a.start : b.start;
  set.sorted = first ? a.sorted : b.sorted;
  return i >= 0 && i < set.n;
}

// Every workgroup forms the grid from the box partials itself (they are few,
// and a launch of its own would cost more than all of them reading them); the
// first one keeps it for the passes that follow.
__global__ __launch_bounds__(256) void k_bin_count(BinSet a, BinSet b, int64_t b0,
                                                   const Box* part, int n_part,
                                                   double cell_size, int64_t cap, Grid* keep) {
  __shared__ Box sh[4];
  __shared__ Grid sg;
  const int64_t n_threads = b0 + b.n;
  int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, i = 0;
  BinSet set;
  bool any = bin_pick(a, b, b0, t, set, i);
  double x[3] = {0.0, 0.0, 0.0};
  // the first point is requested before the box is formed
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (any) x[c] = set.x[c * set.n + i];
  Box box;
  box.clear();
  if ((int)threadIdx.x < n_part) box = part[threadIdx.x];
  box.block_join(sh);
  if (threadIdx.x == 0) {
    sg = make_grid(box, cell_size, cap);
    if (blockIdx.x == 0) *keep = sg;
  }
  __syncthreads();
  const Grid g = sg;
  const double inv = 1.0 / g.cell;
  while (t < n_threads) {
    if (any) {
      const int cx = cell_coord(x[0], g.lo[0], inv, g.dims[0]);
      const int cy = cell_coord(x[1], g.lo[1], inv, g.dims[1]);
      const int cz = cell_coord(x[2], g.lo[2], inv, g.dims[2]);
      const int32_t cid = (cz * g.dims[1] + cy) * g.dims[0] + cx;
      set.cell[i] = cid;
      set.rank[i] = grouped_atomic_add(set.cnt + 1, cid);
    }
    t += (int64_t)gridDim.x * 256;
    any = t < n_threads && bin_pick(a, b, b0, t, set, i);
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (any) x[c] = set.x[c * set.n + i];
  }
}

__global__ __launch_bounds__(256) void k_bin_fill(BinSet a, BinSet b, int64_t b0) {
  BinSet set;
  int64_t i;
  if (!bin_pick(a, b, b0, (int64_t)blockIdx.x * 256 + threadIdx.x, set, i)) return;
  const double* x = set.x;
  const int64_t n = set.n;
  const int32_t pos = set.start[set.cell[i]] + set.rank[i];
  set.sorted[pos] = make_double4(x[i], x[n + i], x[2 * n + i], (double)i);
}

// The fill of few cells (few_cells): the offsets of the sets that the workgroup
// needs are scanned in LDS; the first workgroup keeps them for the passes that
// follow.
__global__ __launch_bounds__(256) void k_bin_scan_fill(BinSet a, BinSet b, int64_t b0,
                                                       const Grid* __restrict__ gp) {
  __shared__ int32_t off[2][kFewCells];
  __shared__ int32_t sums[2][256 / kWave];
  const int tid = threadIdx.x;
  const int64_t t = (int64_t)blockIdx.x * 256;
  BinSet set;
  int64_t i;
  const bool any = bin_pick(a, b, b0, t + tid, set, i);
  double x[3] = {0.0, 0.0, 0.0};
  int32_t cell = 0, rank = 0;
  if (any) {
#pragma unroll
    for (int c = 0; c < 3; ++c) x[c] = set.x[c * set.n + i];
    cell = set.cell[i];
    rank = set.rank[i];
  }
  const int n_cells = (int)gp->n_cells;
  const int per = (n_cells + 255) / 256;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const BinSet& q = s == 0 ? a : b;
    if (blockIdx.x != 0 && !(s == 0 ? t < a.n : t + 256 > b0)) continue;  // uniform
    int32_t sum = 0, total;
    for (int e = tid * per; e < (tid + 1) * per && e < n_cells; ++e) {
      off[s][e] = sum;
      sum += q.cnt[1 + e];
    }
    const int32_t before = block_scan(sum, sums[s], total);
    for (int e = tid * per; e < (tid + 1) * per && e < n_cells; ++e) off[s][e] += before;
    __syncthreads();
    if (blockIdx.x == 0)
      for (int e = tid; e <= n_cells; e += 256) q.start[e] = e < n_cells ? off[s][e] : total;
  }
  if (any)
    set.sorted[off[t + tid < a.n ? 0 : 1][cell] + rank] =
        make_double4(x[0], x[1], x[2], (double)i);
}

// ---------------------------------------------------------------- MP lists
OTM_DEV double sqdist(double ax, double ay, double az, double bx, double by, double bz) {
#pragma clang fp contract(off)
  const double dx = ax - bx, dy = ay - by, dz = az - bz;
  return (dx * dx + dy * dy) + dz * dz;
}

// Visits every node within r of (px,py,pz), in cell order.
template <typename Visit>
OTM_DEV void for_each_neighbor(double px, double py, double pz, double r2, const Grid& g,
                               const int32_t* __restrict__ cell_start,
                               const double4* __restrict__ sorted, Visit&& visit) {
  const double inv = 1.0 / g.cell;
  const int cx = cell_coord(px, g.lo[0], inv, g.dims[0]);
  const int cy = cell_coord(py, g.lo[1], inv, g.dims[1]);
  const int cz = cell_coord(pz, g.lo[2], inv, g.dims[2]);
  for (int z = cz - 1; z <= cz + 1; ++z) {
    if (z < 0 || z >= g.dims[2]) continue;
    for (int y = cy - 1; y <= cy + 1; ++y) {
      if (y < 0 || y >= g.dims[1]) continue;
      const int row = (z * g.dims[1] + y) * g.dims[0];
      const int x0 = cx > 0 ? cx - 1 : 0;
      const int x1 = cx + 1 < g.dims[0] ? cx + 1 : g.dims[0] - 1;
      // cells x0..x1 of one row are contiguous in the sorted array
      const int32_t s0 = cell_start[row + x0], s1 = cell_start[row + x1 + 1];
      for (int32_t s = s0; s < s1; ++s) {
        const double4 nd = sorted[s];
        if (sqdist(px, py, pz, nd.x, nd.y, nd.z) <= r2) visit((int32_t)nd.w);
      }
    }
  }
}

// Row ranges of the 27 cells around cell (cx, cy, cz): the 9 (z, y) rows of
// three cells each are contiguous in the binned array.  Rows outside the
// grid are empty.  pre[k] is the number of candidates before row k.
OTM_DEV void cell_rows(const Grid& g, const int32_t* __restrict__ cell_start, int cx, int cy,
                       int cz, int32_t rs[9], int32_t pre[10]) {
  const int x0 = cx > 0 ? cx - 1 : 0;
  const int x1 = cx + 1 < g.dims[0] ? cx + 1 : g.dims[0] - 1;
  int32_t re[9];
  // branch-free: every load is issued (clamped rows), then masked
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int z = cz - 1 + k / 3, y = cy - 1 + k % 3;
    const bool in = z >= 0 && z < g.dims[2] && y >= 0 && y < g.dims[1];
    const int zc = z < 0 ? 0 : (z >= g.dims[2] ? g.dims[2] - 1 : z);
    const int yc = y < 0 ? 0 : (y >= g.dims[1] ? g.dims[1] - 1 : y);
    const int rw = (zc * g.dims[1] + yc) * g.dims[0];
    const int32_t a = cell_start[rw + x0], b = cell_start[rw + x1 + 1];
    rs[k] = in ? a : 0;
    re[k] = in ? b : 0;
  }
  pre[0] = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) pre[k + 1] = pre[k] + (re[k] - rs[k]);
}

// Position in the binned array of candidate c (0 <= c < pre[9]).
OTM_DEV int32_t cand_pos(int32_t c, const int32_t rs[9], const int32_t pre[10]) {
  int32_t shift = rs[0] - pre[0];
#pragma unroll
  for (int k = 1; k < 9; ++k) shift = c >= pre[k] ? rs[k] - pre[k] : shift;
  return c + shift;
}

OTM_DEV void wave_sync() {
  // the wave's lanes read each other's LDS writes after this point
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

OTM_DEV double lane_value(double v, int t) {  // v of lane t (t uniform)
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, t);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), t);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Cell-centric pass: one wave per grid cell.  All MPs of a cell have the same
// 27 candidate cells, so the wave loads the candidates once and keeps them in
// registers, lane l holding candidates l, l + 64, ...  Each MP of the cell
// (binned like the nodes) is then tested against them: a ballot of the hits,
// taken in candidate order, gives each hit its place in the MP's staging
// row.  The row is in stencil order; the compaction sorts it by node id (the
// four lanes of a quad per row, in registers), which costs far fewer
// instructions than sorting each cell's candidates.  The count goes to cnt[p]; rows
// longer than kRowCap are only counted (the compaction re-finds them).  A
// cell with more than kCand candidates takes each MP separately: hits are
// appended to LDS by ballot and rank-sorted.
//
// The cell index is wave-uniform, so a cell's header (MP range, candidate
// rows) comes from scalar loads, and the next cell's header is requested
// before the current cell is processed.  Each XCD strides over its own
// contiguous eighth of the cells (neighbouring cells share that XCD's L2).
constexpr int kCellWaves = 4;
constexpr unsigned kCellBlocks = 8 * 1024;
constexpr int kCand = 320;
constexpr int kCandChunks = kCand / kWave;
constexpr int kRowCap = kRowCapacity;

struct CellHdr {
  int32_t m0, m1;
  int32_t rs[9], pre[10];
};

OTM_DEV CellHdr cell_header(int64_t c, const Grid& g, const int32_t* __restrict__ cell_start,
                            const int32_t* __restrict__ mp_cell_start) {
  CellHdr h;
  h.m0 = mp_cell_start[c];
  h.m1 = mp_cell_start[c + 1];
  const int32_t ci = (int32_t)c;  // cell counts stay below 2^31
  const int cx = ci % g.dims[0];
  const int cy = (ci / g.dims[0]) % g.dims[1];
  const int cz = ci / (g.dims[0] * g.dims[1]);
  cell_rows(g, cell_start, cx, cy, cz, h.rs, h.pre);
  return h;
}

struct CellLds {  // the hits of one MP in the dense path
  int32_t ids[kCand];
};

// Part `part` of 2^split of a cell's MPs.
OTM_DEV void cell_scan_one(const CellHdr& h, int part, int split, double r2,
                           const double4* __restrict__ sorted,
                           const double4* __restrict__ mp_sorted, int32_t* __restrict__ cnt,
                           int32_t* __restrict__ stage, CellLds& L, int lane) {
  const int32_t share = (((h.m1 - h.m0 + (1 << split) - 1) >> split) + 3) & ~3;
  const int32_t m0 = h.m0 + part * share;
  const int32_t m1 = m0 + share < h.m1 ? m0 + share : h.m1;
  if (m0 >= m1) return;
  const int32_t T = h.pre[9];
  if (T <= kCand) {
    const int nch = (T + kWave - 1) / kWave;  // uniform
    double4 v[kCandChunks];
    // the first 64 MPs of the cell, requested with the candidates
    const int mc0 = m1 - m0 < kWave ? (int)(m1 - m0) : kWave;
    double4 mine = mp_sorted[m0 + (lane < mc0 ? lane : mc0 - 1)];
    // the candidates in stencil order: the rows come out unsorted and the
    // compaction sorts each one by node id
#pragma unroll
    for (int k = 0; k < kCandChunks; ++k) {
      if (k < nch) {
        const int32_t j = k * kWave + lane;
        v[k] = sorted[cand_pos(j < T ? j : 0, h.rs, h.pre)];
      }
    }
    // per chunk: lanes holding a real candidate, and the candidate ids
    bool valid[kCandChunks];
    int32_t cid[kCandChunks];
#pragma unroll
    for (int k = 0; k < kCandChunks; ++k) {
      valid[k] = k * kWave + lane < T;
      cid[k] = (int32_t)v[k].w;
    }
    // NM MPs of the cell (lanes t .. t + NM - 1 of ``mine``) tested together:
    // their chains are independent, so the hardware overlaps them
    auto test_mps = [&](auto nm_tag, int t, int32_t pl) {
      constexpr int NM = decltype(nm_tag)::value;
      double px[NM], py[NM], pz[NM];
      int32_t* row[NM];
      int32_t p[NM];
      uint32_t n[NM];
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        px[i] = lane_value(mine.x, t + i);
        py[i] = lane_value(mine.y, t + i);
        pz[i] = lane_value(mine.z, t + i);
        p[i] = __builtin_amdgcn_readlane(pl, t + i);
        row[i] = stage + (int64_t)p[i] * kRowCap;
        n[i] = 0;
      }
#pragma unroll
      for (int k = 0; k < kCandChunks; ++k) {
        if (k < nch) {
#pragma unroll
          for (int i = 0; i < NM; ++i) {
            // every lane computes the distance (stand-ins are masked), so no
            // branch around it
            const bool hit = (sqdist(px[i], py[i], pz[i], v[k].x, v[k].y, v[k].z) <= r2) &
                             valid[k];
            const uint64_t m = __ballot(hit);
            const uint32_t pos = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, n[i]));
            if (hit & (pos < (uint32_t)kRowCap)) row[i][pos] = cid[k];
            n[i] += (uint32_t)__popcll(m);
          }
        }
      }
      if (lane == 0) {
#pragma unroll
        for (int i = 0; i < NM; ++i) cnt[p[i]] = (int32_t)n[i];
      }
    };
    for (int32_t mb = m0; mb < m1; mb += kWave) {
      const int mc = m1 - mb < kWave ? (int)(m1 - mb) : kWave;
      if (mb != m0) mine = mp_sorted[mb + (lane < mc ? lane : mc - 1)];
      const int32_t pl = (int32_t)mine.w;  // this lane's MP
      int t = 0;
      for (; t + 3 < mc; t += 4) test_mps(std::integral_constant<int, 4>{}, t, pl);
      if (t + 1 < mc) { test_mps(std::integral_constant<int, 2>{}, t, pl); t += 2; }
      if (t < mc) test_mps(std::integral_constant<int, 1>{}, t, pl);
    }
  } else {
    // dense neighbourhood: one MP at a time, candidates read from memory
    for (int32_t m = m0; m < m1; ++m) {
      const double4 mp = mp_sorted[m];
      const int64_t p = (int64_t)mp.w;
      int32_t n = 0;
      for (int32_t b = 0; b < T; b += kWave) {
        const int32_t j = b + lane;
        const double4 nd = sorted[cand_pos(j < T ? j : 0, h.rs, h.pre)];
        const bool hit = j < T && sqdist(mp.x, mp.y, mp.z, nd.x, nd.y, nd.z) <= r2;
        const uint64_t msk = __ballot(hit);
        const int pos = n + (int)__builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(msk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)msk, 0u));
        if (hit && pos < kCand) L.ids[pos] = (int32_t)nd.w;
        n += __popcll(msk);
      }
      wave_sync();
      if (n <= kRowCap) {
        int32_t* row = stage + p * kRowCap;
        if (lane < n) {
          const int32_t id = L.ids[lane];
          int rk = 0;
          for (int t = 0; t < n; ++t) rk += L.ids[t] < id;
          row[rk] = id;
        }
      }
      if (lane == 0) cnt[p] = n;
      wave_sync();
    }
  }
}

// A wave's item is a cell, or with fewer than kMinItems cells (a small body,
// whose cells alone would leave most of the chip idle and their MPs to one
// wave's serial loop) one of up to 2^kMaxSplit parts of a cell's MPs: 4096 MPs
// 9.8 us, 22 whole; 27.6k MPs 17, 28 whole.  Above kMinItems cells the chip is
// full and a part would only fetch its cell's nodes again.
constexpr int kMinItems = 4096;
constexpr int kMaxSplit = 3;

__global__ __launch_bounds__(kCellWaves * kWave) void k_cell_scan(
    double r2, const Grid* __restrict__ gp, int64_t cap_cells,
    const int32_t* __restrict__ cell_start, const double4* __restrict__ sorted,
    const int32_t* __restrict__ mp_cell_start, const double4* __restrict__ mp_sorted,
    int32_t* __restrict__ cnt, int32_t* __restrict__ stage) {
  __shared__ CellLds lds[kCellWaves];
  // wave index as a uniform value, so the cell loop runs on scalar registers
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = (int)(threadIdx.x % kWave);
  const Grid g = *gp;
  const int32_t n_cells = (int32_t)(g.n_cells < cap_cells ? g.n_cells : cap_cells);
  int split = 0;  // 2^split parts
  while (split < kMaxSplit && (n_cells << split) < kMinItems) ++split;
  const int32_t n_items = n_cells << split;  // cells, or under 2 kMinItems
  const int32_t per_xcd = (n_items + 7) / 8;
  const int32_t c_lo = (int32_t)(blockIdx.x % 8u) * per_xcd;
  const int32_t c_hi = c_lo + per_xcd < n_items ? c_lo + per_xcd : n_items;
  const int32_t stride = (int32_t)(gridDim.x / 8u) * kCellWaves;
  int64_t c = (int64_t)c_lo + (int64_t)(blockIdx.x / 8u) * kCellWaves + w;
  if (c >= c_hi) return;
  CellHdr h = cell_header((int32_t)c >> split, g, cell_start, mp_cell_start);
  for (; c < c_hi; c += stride) {
    const int64_t cn = c + stride < c_hi ? c + stride : c;
    // next item's cell, early
    const CellHdr hn = cell_header((int32_t)cn >> split, g, cell_start, mp_cell_start);
    cell_scan_one(h, (int32_t)c & ((1 << split) - 1), split, r2, sorted, mp_sorted, cnt, stage,
                  lds[w], lane);
    h = hn;
  }
}

// Pairs before each run of kPairRun MPs, and before each group of kScanMPs MPs
// within its run (the compaction scans a group's counts itself).  The last
// workgroup to finish scans the runs' totals and reports them to diag.
constexpr int kScanMPs = 64;       // MPs per compaction workgroup
constexpr int kPairRun = 16384;    // MPs per workgroup here, 16 per thread: the
                                   // tickets of smaller runs queue (6M MPs: 63 us
                                   // with runs of 4096, 25 with these)
// Up to here the compaction sums the counts: eight 16-byte loads a thread, in
// flight together (the compaction of 4096 MPs takes 5.6 us with them; the run
// pass alone would take 6).
constexpr int kDirectMPs = 8192;
struct PairRun {
  int64_t pairs;  // of the run, then before it
  int64_t most;   // largest count of the run
};

// Four counts from i on, zero past n.  (The load may reach past the counts,
// within the 256-byte unit of the workspace that ends them.)
OTM_DEV int4 load_counts(const int32_t* __restrict__ cnt, int64_t i, int64_t n) {
  int4 v = i < n ? reinterpret_cast<const int4*>(cnt)[i / 4] : make_int4(0, 0, 0, 0);
  v.y = i + 1 < n ? v.y : 0;
  v.z = i + 2 < n ? v.z : 0;
  v.w = i + 3 < n ? v.w : 0;
  return v;
}

OTM_DEV int32_t wave_max(int32_t m) {
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const int32_t u = __shfl_xor(m, o);
    m = u > m ? u : m;
  }
  return m;
}

__global__ __launch_bounds__(1024) void k_pair_runs(const int32_t* __restrict__ cnt, int64_t n_mp,
                                                    int64_t* __restrict__ group, PairRun* runs,
                                                    int32_t* ticket, int64_t capacity,
                                                    otm_diag* diag) {
  __shared__ int64_t sh[1024 / kWave];
  __shared__ int32_t shm[1024 / kWave];
  __shared__ bool last;
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kPairRun + (int64_t)tid * 16;
  int32_t m = 0;
  int64_t sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int4 c = load_counts(cnt, base + 4 * k, n_mp);
    m = max(m, max(max(c.x, c.y), max(c.z, c.w)));
    sum += ((int64_t)c.x + c.y) + ((int64_t)c.z + c.w);
  }
  m = wave_max(m);
  if (tid % kWave == 0) shm[tid / kWave] = m;
  int64_t total;
  int64_t before = block_scan(sum, sh, total);
  if (tid % (kScanMPs / 16) == 0 && base < n_mp) group[base / kScanMPs] = before;
  if (tid == 0) {
    int32_t most = 0;
    for (int w = 0; w < 1024 / kWave; ++w) most = max(most, shm[w]);
    // seen by the last workgroup through the ticket's release and acquire
    __hip_atomic_store(&runs[blockIdx.x].pairs, total, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&runs[blockIdx.x].most, (int64_t)most, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
           (int32_t)gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  int64_t run = 0;
  m = 0;
  for (int64_t r0 = 0; r0 < gridDim.x; r0 += 1024) {
    const int64_t r = r0 + tid;
    int64_t v = 0;
    if (r < gridDim.x) {
      v = __hip_atomic_load(&runs[r].pairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      m = max(m, (int32_t)__hip_atomic_load(&runs[r].most, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT));
    }
    before = block_scan(v, sh, total);
    if (r < gridDim.x) runs[r].pairs = run + before;
    run += total;
    __syncthreads();
  }
  m = wave_max(m);
  if (tid % kWave == 0) shm[tid / kWave] = m;
  __syncthreads();
  if (tid != 0) return;
  runs[gridDim.x].pairs = run;
  if (diag == nullptr) return;
  for (int w = 0; w < 1024 / kWave; ++w) m = max(m, shm[w]);
  diag->pairs_needed = run;
  diag->max_support = m;
  if (run > capacity) atomicOr(&diag->flags, 1u << (-OTM_ERR_CAPACITY - 1));
}

// Loads lane l's ids of a staged row (16-byte aligned) of K <= 4 PER ids:
// slots PER l and on, those past K INT32_MAX.  Only 16-byte pieces that hold
// ids are read.
template <int PER>
OTM_DEV void load_row_quad(int32_t (&a)[PER], const int32_t* __restrict__ row, int K, int l) {
  const int4* __restrict__ row4 = reinterpret_cast<const int4*>(row);
#pragma unroll
  for (int q = 0; q < PER / 4; ++q) {
    const int e = PER * l + 4 * q;
    int4 v = e < K ? row4[e / 4] : make_int4(INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX);
    a[4 * q] = v.x;
    a[4 * q + 1] = e + 1 < K ? v.y : INT32_MAX;
    a[4 * q + 2] = e + 2 < K ? v.z : INT32_MAX;
    a[4 * q + 3] = e + 3 < K ? v.w : INT32_MAX;
  }
}

// Ascending order of 4 PER ids held by the four lanes of a quad: a bitonic
// network, lane l of the quad holding slots PER l and on.  Compare-exchanges
// between slots PER or 2 PER apart pair a lane with the quad lane l ^ 1 or
// l ^ 2 (DPP quad permutations); the others stay in the lane.
template <int PER>
OTM_DEV void sort_row_quad(int32_t (&a)[PER], int l) {
#pragma unroll
  for (int k = 2; k <= 4 * PER; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= PER) {
        const bool lower = (l & (j / PER)) == 0;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
          const int32_t w = j == PER ? dpp_move<0xB1>(a[e]) : dpp_move<0x4E>(a[e]);
          const int32_t lo = a[e] < w ? a[e] : w, hi = a[e] < w ? w : a[e];
          const bool up = ((PER * l + e) & k) == 0;
          a[e] = lower == up ? lo : hi;
        }
      } else {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
          const int f = e ^ j;
          if (f > e) {
            const int32_t x = a[e], y = a[f];
            const int32_t lo = x < y ? x : y, hi = x < y ? y : x;
            const bool up = ((PER * l + e) & k) == 0;
            a[e] = up ? lo : hi;
            a[f] = up ? hi : lo;
          }
        }
      }
    }
  }
}

// The ids of one row, sorted, at dst (its first id) and on.
template <int PER>
OTM_DEV void put_row_quad(const int32_t (&a)[PER], int32_t* dst, int K, int l) {
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (PER * l + e < K) dst[PER * l + e] = a[e];
}

// Row starts and lists.  A workgroup takes 64 MPs, each of its waves 16 of
// their rows, a quad of lanes per row: the quad loads the staged row, sorts
// it in registers and writes it to the wave's image of its CSR segment in
// LDS, which leaves with unit-stride stores.  Every wave scans the 64 counts
// itself, so that the waves need not wait for one another.  Rows longer than
// kRowCap are found again and sorted in place by one lane.  The pairs before
// a workgroup are those before its run plus its group's place in the run; for
// up to kDirectMPs MPs (DIRECT) it sums the counts itself instead, which
// spares the run pass, and the first workgroup reports the totals to diag.
//
// Bound by memory: 1.13M MPs, 27 ids each, 60 us (a pass that loaded whole
// rows of kRowCap ids to LDS, sorted them there and marked the MP of each
// output element 90 us); lists to 1.1 times the radius, with
// many rows past 32 ids, 101 us (776 with those rows sorted by insertion).
template <bool DIRECT>
__global__ __launch_bounds__(256) void k_nbr_compact(
    const double* __restrict__ xp, int64_t n_mp, double r2, const Grid* __restrict__ gp,
    const int32_t* __restrict__ cell_start, const double4* __restrict__ sorted,
    const int32_t* __restrict__ cnt, const int64_t* __restrict__ group,
    const PairRun* __restrict__ runs, int64_t n_runs, int64_t* __restrict__ offsets,
    const int32_t* __restrict__ stage, int64_t capacity, int32_t* __restrict__ idx,
    otm_diag* diag) {
  static_assert(kScanMPs == kWave && kPairRun % kScanMPs == 0, "one count per lane");
  static_assert(kRowCap % 4 == 0 && kRowCap <= 64, "whole 16-byte pieces, at most 64 slots");
  constexpr int kWaveRows = kScanMPs / 4;
  __shared__ int32_t image[4][kWaveRows * kRowCap];
  const int tid = threadIdx.x, lane = tid % kWave, l = tid % 4;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int64_t blk = xcd_block();
  const int64_t p0 = blk * kScanMPs;
  if (p0 >= n_mp) return;
  const int nloc = (int)(n_mp - p0 < kScanMPs ? n_mp - p0 : kScanMPs);
  const int32_t mine = lane < nloc ? cnt[p0 + lane] : 0;
  int64_t start, total_pairs;
  if (!DIRECT) {
    start = runs[p0 / kPairRun].pairs + group[blk];
    total_pairs = runs[n_runs].pairs;
  }
  const int i = kWaveRows * w + lane / 4;  // this quad's row
  const int32_t K = __shfl(mine, i);
  const int32_t staged = K <= kRowCap ? K : 0;
  const int32_t* __restrict__ row = stage + (p0 + i) * kRowCap;
  const bool wide = __ballot(staged > 32) != 0;
  int32_t a[8];
  if (!wide) load_row_quad<8>(a, row, staged, l);
  if (DIRECT) {
    __shared__ int64_t sum_before[4], sum_all[4];
    __shared__ int32_t most_of[4];
    int64_t before = 0, all = 0;
    int32_t most = 0;
#pragma unroll
    for (int k = 0; k < kDirectMPs / 1024; ++k) {
      const int64_t q = (k * 256 + tid) * 4;
      const int4 v = load_counts(cnt, q, n_mp);
      const int32_t c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        all += c[e];
        before += q + e < p0 ? c[e] : 0;
        most = max(most, c[e]);
      }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
      before += __shfl_xor(before, o);
      all += __shfl_xor(all, o);
    }
    most = wave_max(most);
    if (lane == 0) {
      sum_before[w] = before;
      sum_all[w] = all;
      most_of[w] = most;
    }
    __syncthreads();
    start = (sum_before[0] + sum_before[1]) + (sum_before[2] + sum_before[3]);
    total_pairs = (sum_all[0] + sum_all[1]) + (sum_all[2] + sum_all[3]);
    if (blk == 0 && tid == 0 && diag != nullptr) {
      diag->pairs_needed = total_pairs;
      diag->max_support = max(max(most_of[0], most_of[1]), max(most_of[2], most_of[3]));
      if (total_pairs > capacity) atomicOr(&diag->flags, 1u << (-OTM_ERR_CAPACITY - 1));
    }
  }
  int64_t excl = mine;  // pairs of the group before this lane's MP
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t u = __shfl_up(excl, o);
    excl += lane >= o ? u : 0;
  }
  if (w == 0) {
    if (lane < nloc) offsets[p0 + lane] = start + excl - mine;
    if (lane == nloc - 1 && p0 + nloc == n_mp) offsets[n_mp] = start + excl;
  }
  if (total_pairs > capacity) return;  // lists do not fit: row starts only
  excl -= mine;
  const int64_t seg = start + __shfl(excl, kWaveRows * w);  // the wave's first pair
  const int64_t o = start + __shfl(excl, i);                // the row's
  // image of the wave's segment; with a row past kRowCap, straight to memory
  const bool fits = __ballot(K > kRowCap) == 0;
  int32_t* img = image[w];
  if (!wide) {
    sort_row_quad<8>(a, l);
    if (fits) put_row_quad<8>(a, img + (int)(o - seg), staged, l);
    else put_row_quad<8>(a, idx + o, staged, l);
  } else {
    int32_t b[16];
    load_row_quad<16>(b, row, staged, l);
    sort_row_quad<16>(b, l);
    if (fits) put_row_quad<16>(b, img + (int)(o - seg), staged, l);
    else put_row_quad<16>(b, idx + o, staged, l);
  }
  if (fits) {
    const int total = (int)(__shfl(o, kWave - 1) - seg) + __shfl(K, kWave - 1);
    // one wave writes and reads the image: its LDS accesses run in order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int e = lane; e < total; e += kWave) idx[seg + e] = img[e];
    return;
  }
  // long supports
  if (l == 0 && K > kRowCap) {
    const int64_t p = p0 + i;
    const Grid g = *gp;
    int32_t n = 0;
    for_each_neighbor(xp[p], xp[n_mp + p], xp[2 * n_mp + p], r2, g, cell_start, sorted,
                      [&](int32_t id) {
                        int32_t j = n++;
                        while (j > 0 && idx[o + j - 1] > id) {
                          idx[o + j] = idx[o + j - 1];
                          --j;
                        }
                        idx[o + j] = id;
                      });
  }
}

// No MPs: one row start and nothing found.
__global__ void k_search_empty(int64_t* offsets, otm_diag* diag) {
  offsets[0] = 0;
  if (diag != nullptr) {
    diag->pairs_needed = 0;
    diag->max_support = 0;
  }
}

void launch_search(int64_t n_nodes, const double* x_nodes, int64_t n_mp, const double* x_mp,
                   double r_list, double cell_size, int64_t pair_capacity, int64_t* nbr_offsets,
                   int32_t* nbr_idx, const Workspace& w, otm_diag* diag, hipStream_t s,
                   bool boxed) {
  if (n_mp <= 0) {
    k_search_empty<<<1, 1, 0, s>>>(nbr_offsets, diag);
    return;
  }
  const BinCounters z = bin_counters(w, n_mp);
  Box* part = reinterpret_cast<Box*>(w.bbox_part);
  unsigned n_part = (unsigned)((n_nodes + 255) / 256);
  if (!boxed) {
    n_part = bbox_blocks(n_nodes);
    k_bbox_partial<<<n_part, 256, 0, s>>>(x_nodes, n_nodes, part, z);
  }
  // nodes and MPs binned on the grid together: one count, one two-array scan,
  // one fill.  The MPs' ranks lie where their rows are staged later.
  const BinSet nodes{x_nodes, n_nodes, w.node_cell, w.node_rank, z.node_cnt, w.cell_start,
                     w.sorted};
  const BinSet mps{x_mp, n_mp, w.mp_cell, w.stage, z.mp_cnt, w.mp_cell_start, w.mp_sorted};
  const int64_t b0 = (n_nodes + kWave - 1) / kWave * kWave;
  const int64_t nt = b0 + n_mp;
  const unsigned nbt = (unsigned)((nt + 255) / 256);
  k_bin_count<<<nbt < kCountBlocks ? nbt : kCountBlocks, 256, 0, s>>>(
      nodes, mps, b0, part, (int)n_part, cell_size, w.cap_cells, w.grid);
  if (few_cells(w, n_mp)) {
    k_bin_scan_fill<<<nbt, 256, 0, s>>>(nodes, mps, b0, w.grid);
  } else {
    scan_impl<int32_t>(w.cell_start + 1, w.mp_cell_start + 1, w.cap_cells, w.scan_aux,
                       &w.grid->n_cells, s);
    k_bin_fill<<<nbt, 256, 0, s>>>(nodes, mps, b0);
  }
  const double r2 = r_list * r_list;
  // a fixed grid (a multiple of the 8 XCDs) strides over the items.  The MPs'
  // cells are not needed any more: their counts take that place.
  const int64_t most = w.cap_cells > 2 * kMinItems ? w.cap_cells : 2 * kMinItems;
  const int64_t want = (most + kCellWaves - 1) / kCellWaves;
  const unsigned cells = want < kCellBlocks ? (unsigned)((want + 7) / 8 * 8) : kCellBlocks;
  int32_t* cnt = w.mp_cell;
  k_cell_scan<<<cells, kCellWaves * kWave, 0, s>>>(r2, w.grid, w.cap_cells, w.cell_start,
                                                   w.sorted, w.mp_cell_start, w.mp_sorted, cnt,
                                                   w.stage);
  const unsigned nbs = (unsigned)((n_mp + kScanMPs - 1) / kScanMPs);
  if (n_mp <= kDirectMPs) {
    k_nbr_compact<true><<<nbs, 256, 0, s>>>(x_mp, n_mp, r2, w.grid, w.cell_start, w.sorted, cnt,
                                            nullptr, nullptr, 0, nbr_offsets, w.stage,
                                            pair_capacity, nbr_idx, diag);
    return;
  }
  // the binned MPs are not needed any more either: the runs' totals and the
  // groups' places, which are far smaller, take their place
  const int64_t n_runs = (n_mp + kPairRun - 1) / kPairRun;
  PairRun* runs = reinterpret_cast<PairRun*>(w.mp_sorted);
  int64_t* group = reinterpret_cast<int64_t*>(runs + n_runs + 1);
  k_pair_runs<<<(unsigned)n_runs, 1024, 0, s>>>(cnt, n_mp, group, runs, w.ticket, pair_capacity, diag);
  k_nbr_compact<false><<<nbs, 256, 0, s>>>(x_mp, n_mp, r2, w.grid, w.cell_start, w.sorted, cnt,
                                           group, runs, n_runs, nbr_offsets, w.stage,
                                           pair_capacity, nbr_idx, diag);
}

}  // namespace otm

// Exact k nearest neighbours through a uniform grid (the same lists as a
// search over all points: float32 squared distance ((dx*dx + dy*dy) + dz*dz),
// every operation rounded, ties by index), followed by the FP64
// neighbourhood covariance and curvature (Sec. III-A).
//
// 1. The grid (grid_small_kernel: one block, cells in LDS; or the grid_*
//    kernels for large clouds): the bounding box of the finite points, a trial
//    cell of two points per cell of the box, the occupancy of the trial
//    cells, and the final cell for about grid_occ(k) points per occupied cell;
//    then a counting sort of the points by cell.  The order inside a cell
//    does not matter because candidates are ranked by the (distance, index)
//    key, and neither does the cell size.
// 2. knn_kernel: 16 lanes per query, queries in cell order.  The points of
//    the 27 cells around the query's are read row by row (the cells of a
//    row are adjacent in the sorted array, so a row is one span), and those
//    nearer than every unsearched cell go to the query's list in LDS; k of
//    them are the answer.  Where the query's own cell already holds k points
//    (the dense parts of a depth frame), it is searched first and its k-th
//    key limits the rows and cells of the rest; where the 27 cells hold k
//    points but not near enough, their k-th key limits a second ring.  The
//    list is ranked by counting (every lane counts the keys below its own),
//    which needs neither a sorting network nor a register list.
// 3. knn_far_kernel: the queries left over.  One wave per outlier in empty
//    space, which looks at growing rings of cells and then at the blocks of
//    8 x 8 x 8 cells that hold points.
//
// What bounds it: the number of candidates (about 11 occupied cells of a
// surface) and the latency of three dependent loads per query, which many
// small queries per CU hide.  One lane per query, as before, kept a sorted
// list in registers and left a 1 024-point cloud on four CUs and a
// 36 000-point one on 141.  Both search kernels, before and now:
//    1 024 points, k = 24:    94 us,   23 us
//   36 000 points, k = 24:   425 us,   77 us
//  307 200 points, k = 16: 1 561 us,  355 us
// and the build of the last, 600 us and 52 us (its cell scan was one block's).
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "grid_geom.h"
#include "launch.h"

namespace sgr {

// Workspace and arrays of one cloud's search.
struct GridJob {
  const float* x;
  const float* y;
  const float* z;
  float* a_out;     // curvatures, or nullptr
  int n, max_cells;
  float occ;        // wanted occupancy (mean over the points of their cell's count)
  float reach;      // cells up to twice smaller than this are made as large (0: none)
  GridInfo* gi;
  int* cell_of;     // [n] (packed)
  int* rank;        // [n] rank of the point within its cell
  int* counts;      // [max_cells]
  int* starts;      // [max_cells + 1]
  int* part;        // per-block partials of the large build (GRID_PART ints)
  float4* spts;     // points in cell order, w = index
  int* scell;       // their cells' coordinates, packed (pack_cell)
  float4* p4;       // points in their own order, (x, y, z, 0)
  int32_t* nbr;     // neighbour lists
  int* blocks;      // [0] number of blocks of BLK^3 cells that hold points, then those (pack_cell)
};

// One job by value (one cloud), or a table of jobs and a (cloud, block) list.
struct GridArgs {
  GridJob one;
  const GridJob* jobs;
  const int2* bmap;
};

// The job of this block and the block's number within it; pointers marked as
// global memory (gptr).
__device__ inline GridJob job_of(const GridArgs& A, int& block, int* cloud = nullptr) {
  int c = 0;
  block = blockIdx.x;
  if (A.jobs) {
    const int2 cb = A.bmap[blockIdx.x];
    c = cb.x;
    block = cb.y;
  }
  if (cloud) *cloud = c;
  GridJob J = A.jobs ? A.jobs[c] : A.one;
  J.x = gptr(J.x), J.y = gptr(J.y), J.z = gptr(J.z), J.a_out = gptr(J.a_out), J.gi = gptr(J.gi);
  J.cell_of = gptr(J.cell_of), J.rank = gptr(J.rank), J.counts = gptr(J.counts), J.starts = gptr(J.starts);
  J.part = gptr(J.part), J.spts = gptr(J.spts), J.scell = gptr(J.scell), J.p4 = gptr(J.p4), J.nbr = gptr(J.nbr);
  J.blocks = gptr(J.blocks);
  return J;
}
__device__ inline GridJob job_at(const GridArgs& A, int c) {
  GridJob J = A.jobs ? A.jobs[c] : A.one;
  J.gi = gptr(J.gi), J.starts = gptr(J.starts), J.spts = gptr(J.spts), J.scell = gptr(J.scell), J.nbr = gptr(J.nbr);
  J.blocks = gptr(J.blocks);
  return J;
}

// The grid of a block's job in scalar registers (loaded through a pointer it is
// not known to be the same in every lane).
__device__ inline GridInfo block_grid(const GridInfo* gi) {
  static_assert(sizeof(GridInfo) % 4 == 0, "whole words");
  union {
    GridInfo G;
    int w[sizeof(GridInfo) / 4];
  } u{*gi};
  for (int e = 0; e < (int)(sizeof(GridInfo) / 4); ++e) u.w[e] = __builtin_amdgcn_readfirstlane(u.w[e]);
  return u.G;
}

// ------------------------------------------------------------------- grid
// Wanted occupancy for k neighbours.  Counted over surfaces of even
// density, a query of occupancy 0.45 k finds twice k points within the distance its 27 cells
// cover, among five times k candidates, and one in fifty finds fewer than k;
// at 0.3 k it is one in four, at 0.7 k the candidates are nine times k.
inline float grid_occ(int k) { return std::max(2.0f, 0.5f * (float)k); }

// Box of the finite points among the block's (points base + tid, stride):
// an infinite coordinate would make the grid one row of cells.
template <int BT>
__device__ inline void box_of(const GridJob& J, int first, int stride, float box[6], float* lds) {
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll 4
  for (int i = first + threadIdx.x; i < J.n; i += stride) {
    const float p[3] = {J.x[i], J.y[i], J.z[i]};
    const bool fin = isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]);
    for (int a = 0; a < 3; ++a) {
      v[a] = fminf(v[a], fin ? p[a] : INFINITY);
      v[3 + a] = fmaxf(v[3 + a], fin ? p[a] : -INFINITY);
    }
  }
  for (int a = 0; a < 6; ++a) {
    float m = a < 3 ? v[a] : -v[a];
    m = fminf(m, __shfl_xor(m, 32, 64));
    m = fminf(m, __shfl_xor(m, 16, 64));
    m = fminf(m, __uint_as_float(xor_lane_u<8>(__float_as_uint(m))));
    m = fminf(m, __uint_as_float(xor_lane_u<4>(__float_as_uint(m))));
    m = fminf(m, __uint_as_float(xor_lane_u<2>(__float_as_uint(m))));
    m = fminf(m, __uint_as_float(xor_lane_u<1>(__float_as_uint(m))));
    if ((threadIdx.x & 63) == 0) lds[(threadIdx.x >> 6) * 6 + a] = m;
  }
  __syncthreads();
  for (int a = 0; a < 6; ++a) {
    float m = lds[a];
    for (int w = 1; w < BT / 64; ++w) m = fminf(m, lds[w * 6 + a]);
    box[a] = a < 3 ? m : -m;
  }
  __syncthreads();
}

// Exclusive scan of one int per thread over a block of BT threads; returns
// the prefix, total receives the sum.  lds: BT / 64 ints.
template <int BT>
__device__ inline int block_scan(int v, int& total, int* lds) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(x, off, 64);
    if (lane >= off) x += o;
  }
  if (lane == 63) lds[w] = x;
  __syncthreads();
  int before = 0;
  total = 0;
  for (int u = 0; u < BT / 64; ++u) {
    if (u < w) before += lds[u];
    total += lds[u];
  }
  __syncthreads();
  return before + x - v;
}

// Lists block number b of the grid (wave-uniform) if it holds points; lane l
// looks at one of its BLK^2 rows of cells.  start(c): first point of cell c.
template <class Start>
__device__ inline void list_block(const GridInfo& G, int b, int* blocks, Start&& start) {
  const int bd0 = (G.dims[0] + BLK - 1) / BLK, bd1 = (G.dims[1] + BLK - 1) / BLK;
  const int bc[3] = {b % bd0, b / bd0 % bd1, b / (bd0 * bd1)};
  const int lane = threadIdx.x & 63;
  const int cy = bc[1] * BLK + lane % BLK, cz = bc[2] * BLK + lane / BLK;
  bool any = false;
  if (cy < G.dims[1] && cz < G.dims[2]) {
    const int row = (cz * G.dims[1] + cy) * G.dims[0];
    any = start(row + min(G.dims[0], bc[0] * BLK + BLK)) > start(row + bc[0] * BLK);
  }
  if (__any(any) && lane == 0) blocks[1 + atomicAdd(blocks, 1)] = pack_cell(G, bc);
}
// Whole grid of one cloud in one block, its cells in LDS as 16-bit halves (so
// n <= 65 535): one launch and no global atomics where the points are few
// (the phases of the large build are launches of 3 to 5 us each, whatever the
// size).
constexpr int SM_BT = 1024;
constexpr int SM_WORDS = 36 * SM_BT;  // 144 KB of the CU's 160 KB of LDS, two cells a word

__device__ inline int half_of(int w, int c) { return c & 1 ? (int)((unsigned)w >> 16) : w & 0xffff; }

__global__ __launch_bounds__(SM_BT) void grid_small_kernel(GridArgs A, int2* __restrict__ far) {
  extern __shared__ int s_cnt[];  // [(max_cells + 1) / 2]
  __shared__ float s_box[(SM_BT / 64) * 6];
  __shared__ int s_scan[SM_BT / 64];
  __shared__ double s_red[SM_BT / 64];
  __shared__ GridInfo s_g;
  int b, cloud;
  const GridJob J = job_of(A, b, &cloud);
  const int tid = threadIdx.x;
  if (cloud == 0 && tid == 0) far[0] = make_int2(0, 0);  // queries left to the far pass
  if (tid == 0) J.blocks[0] = 0;
  float box[6];
  box_of<SM_BT>(J, 0, SM_BT, box, s_box);
  if (tid == 0) s_g = grid_trial(box, J.n, J.max_cells);
  __syncthreads();
  GridInfo G = s_g;
  for (int pass = 0; pass < 2; ++pass) {
    // counts of the trial cells, then of the final ones
    const int words = (G.ncells + 1) >> 1;
    for (int w = tid; w < words; w += SM_BT) s_cnt[w] = 0;
    __syncthreads();
#pragma unroll 4
    for (int i = tid; i < J.n; i += SM_BT) {
      const int c = cell_index(G, J.x[i], J.y[i], J.z[i]);
      atomicAdd(&s_cnt[c >> 1], c & 1 ? 1 << 16 : 1);
    }
    __syncthreads();
    if (pass) break;
    double sq[1] = {0.0};
    for (int w = tid; w < words; w += SM_BT) {
      const double lo = (double)half_of(s_cnt[w], 0), hi = (double)half_of(s_cnt[w], 1);
      sq[0] += lo * lo + hi * hi;
    }
    block_sum<1, SM_BT>(sq, s_red);
    if (tid == 0) {
      grid_resize(s_g, sq[0] / (double)J.n, J.occ, J.reach, J.max_cells);
      *J.gi = s_g;
    }
    __syncthreads();
    G = s_g;
  }
  // exclusive scan in place: each thread a run of words
  const int words = (G.ncells + 1) >> 1;
  const int per = (words + SM_BT - 1) / SM_BT;
  const int w0 = min(words, tid * per), w1 = min(words, w0 + per);
  int sum = 0;
  for (int w = w0; w < w1; ++w) sum += half_of(s_cnt[w], 0) + half_of(s_cnt[w], 1);
  int total;
  int run = block_scan<SM_BT>(sum, total, s_scan);
  for (int w = w0; w < w1; ++w) {
    const int lo = half_of(s_cnt[w], 0), hi = half_of(s_cnt[w], 1);
    s_cnt[w] = run | (run + lo) << 16;
    run += lo + hi;
  }
  __syncthreads();
  for (int c = tid; c < G.ncells; c += SM_BT) J.starts[c] = half_of(s_cnt[c >> 1], c);
  if (tid == 0) J.starts[G.ncells] = J.n;
  for (int b = tid >> 6; b < block_count(G); b += SM_BT / 64)
    list_block(G, b, J.blocks, [&](int c) { return c < G.ncells ? half_of(s_cnt[c >> 1], c) : J.n; });
  __syncthreads();  // the starts are read above before the scatter moves them
#pragma unroll 4
  for (int i = tid; i < J.n; i += SM_BT) {
    const float x = J.x[i], y = J.y[i], z = J.z[i];
    int cc[3];
    cell_of_point(G, x, y, z, cc);
    const int c = cell_index(G, cc);
    const int pos = half_of(atomicAdd(&s_cnt[c >> 1], c & 1 ? 1 << 16 : 1), c);
    J.spts[pos] = make_float4(x, y, z, __int_as_float(i));
    J.scell[pos] = pack_cell(G, cc);
    J.p4[i] = make_float4(x, y, z, 0.f);
  }
}

// The same in five launches over many blocks.  Partials: LG_BLOCKS boxes of 6
// floats, then LG_BLOCKS (points, occupied) pairs, then the scan's block sums.
constexpr int LG_BT = 256;
constexpr int LG_BLOCKS = 256;
constexpr int LG_SCAN = 4096;  // cells per block of the scan
constexpr int LG_PART = LG_BLOCKS * 8;

// Boxes per block; clears the counts and the far list.
__global__ __launch_bounds__(LG_BT) void grid_box_kernel(GridJob J, int2* __restrict__ far) {
  __shared__ float s_box[(LG_BT / 64) * 6];
  const int t = blockIdx.x * LG_BT + threadIdx.x, nt = gridDim.x * LG_BT;
  if (t == 0) {
    far[0] = make_int2(0, 0);
    J.blocks[0] = 0;
  }
  for (int c = t; c < J.max_cells; c += nt) J.counts[c] = J.starts[c] = 0;
  float box[6];
  box_of<LG_BT>(J, blockIdx.x * LG_BT, nt, box, s_box);
  if (threadIdx.x < 6) reinterpret_cast<float*>(J.part)[blockIdx.x * 6 + threadIdx.x] = box[threadIdx.x];
}

// Box of all blocks' boxes, in every thread.
__device__ inline void box_total(const GridJob& J, int nb, float box[6], float* lds) {
  const float* p = reinterpret_cast<const float*>(J.part);
  float v[6];
  for (int a = 0; a < 6; ++a) v[a] = (int)threadIdx.x < nb ? p[threadIdx.x * 6 + a] : (a < 3 ? INFINITY : -INFINITY);
  for (int a = 0; a < 6; ++a) {
    float m = a < 3 ? v[a] : -v[a];
    for (int off = 32; off > 0; off >>= 1) m = fminf(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) lds[(threadIdx.x >> 6) * 6 + a] = m;
  }
  __syncthreads();
  for (int a = 0; a < 6; ++a) {
    float m = lds[a];
    for (int w = 1; w < LG_BT / 64; ++w) m = fminf(m, lds[w * 6 + a]);
    box[a] = a < 3 ? m : -m;
  }
}

// Lane's run of equal cells among neighbouring points (scan order puts them
// in the same cell often, and atomics of a wave to one address are served one
// by one): first is the run's first lane, len its length (valid there).
__device__ inline bool cell_run(int c, int& first, int& len) {
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(c, 1, 64);
  const bool head = lane == 0 || prev != c;
  const uint64_t heads = __ballot(head);
  const uint64_t upto = ~0ull >> (63 - lane);  // lanes 0 .. lane
  first = 63 - __builtin_clzll(heads & upto);
  const uint64_t after = heads & ~upto;
  len = (after ? __builtin_ctzll(after) : 64) - lane;
  return head;
}

// Occupancy of the trial grid, estimated on one cell in eight (chosen by a
// hash): the points of those cells, and the sum of their counts' squares,
// which grows by (old + len)^2 - old^2 as a run of len points is counted.
__global__ __launch_bounds__(LG_BT) void grid_occupancy_kernel(GridJob J) {
  __shared__ float s_box[(LG_BT / 64) * 6];
  __shared__ GridInfo s_g;
  __shared__ float s_sum[2];
  float box[6];
  box_total(J, LG_BLOCKS, box, s_box);
  if (threadIdx.x == 0) {
    s_g = grid_trial(box, J.n, J.max_cells);
    s_sum[0] = s_sum[1] = 0.f;
  }
  __syncthreads();
  const GridInfo G = s_g;
  float pts = 0.f, sq = 0.f;
  const int nt = gridDim.x * LG_BT;
  for (int base = blockIdx.x * LG_BT; base < J.n; base += nt) {  // whole blocks: every lane takes part
    const int i = base + threadIdx.x;
    const int c = i < J.n ? cell_index(G, J.x[i], J.y[i], J.z[i]) : -1 - (int)(threadIdx.x & 63);
    int first, len;
    if (cell_run(c, first, len) && i < J.n && ((unsigned)c * 2654435761u) >> 29 == 0u) {
      const float old = (float)atomicAdd(&J.starts[c], len);
      pts += (float)len;
      sq += (float)len * (2.f * old + (float)len);
    }
  }
  atomicAdd(&s_sum[0], pts);
  atomicAdd(&s_sum[1], sq);
  __syncthreads();
  if (threadIdx.x < 2)
    reinterpret_cast<float*>(J.part)[LG_BLOCKS * 6 + blockIdx.x * 2 + threadIdx.x] = s_sum[threadIdx.x];
}

// Cell of every point, its count and the point's rank in it.
__global__ __launch_bounds__(LG_BT) void grid_count_kernel(GridJob J) {
  __shared__ float s_box[(LG_BT / 64) * 6];
  __shared__ GridInfo s_g;
  float box[6];
  box_total(J, LG_BLOCKS, box, s_box);
  __syncthreads();
  {
    // LG_BT = LG_BLOCKS partials; the cell size needs no exact sum, but
    // every block has to find the same one: a fixed order
    static_assert(LG_BT == LG_BLOCKS, "one partial per thread");
    const float* p = reinterpret_cast<const float*>(J.part) + LG_BLOCKS * 6;
    float v[2] = {p[2 * threadIdx.x], p[2 * threadIdx.x + 1]};
    for (int e = 0; e < 2; ++e) {
      for (int off = 32; off > 0; off >>= 1) v[e] += __shfl_xor(v[e], off, 64);
      if ((threadIdx.x & 63) == 0) s_box[(threadIdx.x >> 6) * 2 + e] = v[e];
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float pts = 0.f, sq = 0.f;
    for (int w = 0; w < LG_BT / 64; ++w) {
      pts += s_box[2 * w];
      sq += s_box[2 * w + 1];
    }
    GridInfo G = grid_trial(box, J.n, J.max_cells);
    if (pts > 0.f) grid_resize(G, (double)sq / (double)pts, J.occ, J.reach, J.max_cells);
    s_g = G;
    if (blockIdx.x == 0) *J.gi = G;
  }
  __syncthreads();
  const GridInfo G = s_g;
  const int lane = threadIdx.x & 63;
  const int nt = gridDim.x * LG_BT;
  for (int base = blockIdx.x * LG_BT; base < J.n; base += nt) {  // whole blocks: every lane takes part
    const int i = base + threadIdx.x;
    int cc[3] = {0, 0, 0}, c = -1 - lane;
    if (i < J.n) {
      cell_of_point(G, J.x[i], J.y[i], J.z[i], cc);
      c = cell_index(G, cc);
    }
    int first, len, r = 0;
    if (cell_run(c, first, len) && i < J.n) r = atomicAdd(&J.counts[c], len);
    r = __shfl(r, first, 64) + lane - first;
    if (i < J.n) {
      J.cell_of[i] = pack_cell(G, cc);
      J.rank[i] = r;
    }
  }
}

// Exclusive scan of the counts: block sums, then every block adds the sums
// before it.
__global__ __launch_bounds__(1024) void grid_sums_kernel(GridJob J) {
  __shared__ int s_w[16];
  const int nc = J.gi->ncells;
  const int i = blockIdx.x * LG_SCAN + threadIdx.x * 4;
  int v = 0;
  if (i < nc)
    for (int u = 0; u < 4; ++u) v += i + u < nc ? J.counts[i + u] : 0;
  int total;
  (void)block_scan<1024>(v, total, s_w);
  if (threadIdx.x == 0) J.part[LG_PART + blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void grid_starts_kernel(GridJob J) {
  __shared__ int s_w[16];
  const int nc = J.gi->ncells;
  const int first = blockIdx.x * LG_SCAN;
  if (first >= nc) return;
  int before = 0;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += 1024) before += J.part[LG_PART + b];
  int offset;
  (void)block_scan<1024>(before, offset, s_w);
  const int i = first + threadIdx.x * 4;
  int v[4], sum = 0;
  for (int u = 0; u < 4; ++u) {
    v[u] = i + u < nc ? J.counts[i + u] : 0;
    sum += v[u];
  }
  int total;
  int run = offset + block_scan<1024>(sum, total, s_w);
  for (int u = 0; u < 4; ++u) {
    if (i + u < nc) J.starts[i + u] = run;
    run += v[u];
  }
  if (first + LG_SCAN >= nc && threadIdx.x == 0) J.starts[nc] = offset + total;
}

// The first point_blocks blocks move the points, the others list the blocks
// of cells.
__global__ __launch_bounds__(LG_BT) void grid_scatter_kernel(GridJob J, int point_blocks) {
  if ((int)blockIdx.x >= point_blocks) {
    const GridInfo G = *J.gi;
    const int nw = (gridDim.x - point_blocks) * (LG_BT / 64);
    for (int b = (blockIdx.x - point_blocks) * (LG_BT / 64) + (threadIdx.x >> 6); b < block_count(G); b += nw)
      list_block(G, b, J.blocks, [&](int c) { return J.starts[c]; });
    return;
  }
  const int i = blockIdx.x * LG_BT + threadIdx.x;
  if (i >= J.n) return;
  const float x = J.x[i], y = J.y[i], z = J.z[i];
  const GridInfo G = *J.gi;
  const int pc = J.cell_of[i];
  int cc[3];
  unpack_cell(G, pc, cc);
  const int pos = J.starts[cell_index(G, cc)] + J.rank[i];
  J.spts[pos] = make_float4(x, y, z, __int_as_float(i));
  J.scell[pos] = pc;
  J.p4[i] = make_float4(x, y, z, 0.f);
}

// ----------------------------------------------------------------- search
// Keys are (float32 distance bits << 32 | index): for distances >= 0 the bit
// pattern orders like the value, so one unsigned compare gives the (distance,
// index) order.
__device__ inline uint64_t point_key(const float4& P, const float4& q) {
  const float ex = __fsub_rn(P.x, q.x), ey = __fsub_rn(P.y, q.y), ez = __fsub_rn(P.z, q.z);
  const float d2 = __fadd_rn(__fadd_rn(__fmul_rn(ex, ex), __fmul_rn(ey, ey)), __fmul_rn(ez, ez));
  return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)__float_as_int(P.w);
}
// The same with the squares fused into the sums, as a search that is compiled
// with contraction rounds them.
__device__ inline uint64_t point_key_fused(const float4& P, const float4& q) {
  const float ex = __fsub_rn(P.x, q.x), ey = __fsub_rn(P.y, q.y), ez = __fsub_rn(P.z, q.z);
  const float d2 = __builtin_fmaf(ez, ez, __builtin_fmaf(ex, ex, __fmul_rn(ey, ey)));
  return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)__float_as_int(P.w);
}
// LDS written by some lanes of a wave is read by others of the same wave.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Sum of an int over the lanes of a group.
template <int GL>
__device__ inline int group_sum(int v) {
  if constexpr (GL == 64) {
    v += (int)xor_lane_u<32>((unsigned)v);
    v += (int)xor_lane_u<16>((unsigned)v);
  }
  v += (int)xor_lane_u<8>((unsigned)v);
  v += (int)xor_lane_u<4>((unsigned)v);
  v += (int)xor_lane_u<2>((unsigned)v);
  v += (int)xor_lane_u<1>((unsigned)v);
  return v;
}
template <int GL>
__device__ inline unsigned group_max(unsigned v) {
  if constexpr (GL == 64) {
    v = max(v, xor_lane_u<32>(v));
    v = max(v, xor_lane_u<16>(v));
  }
  v = max(v, xor_lane_u<8>(v));
  v = max(v, xor_lane_u<4>(v));
  v = max(v, xor_lane_u<2>(v));
  return max(v, xor_lane_u<1>(v));
}

// A query's list of candidate keys in LDS, kept by a group of GL lanes (GL
// 16 or 64).  Keys not below `bound` are refused.  trim() drops keys that k
// others undercut and lowers the bound, by bisection on the distance bits (a
// few counts of the list) instead of ranking it; the ranks of what is left are
// counted once, at the end.
template <int GL, int CAP>
struct KeyList {
  static constexpr int NE = (CAP + GL - 1) / GL;  // entries of a lane: l, l + GL, ...
  static constexpr int SLACK = 12;                // keys beyond k that trim() may leave
  uint64_t* key;   // [CAP]
  int cnt;
  int k;
  uint64_t bound;

  __device__ void load(uint64_t (&mine)[NE]) const {
    const int l = threadIdx.x % GL;
    wave_sync();
#pragma unroll
    for (int u = 0; u < NE; ++u) mine[u] = l + u * GL < cnt ? key[l + u * GL] : ~0ull;
    wave_sync();
  }

  // rk[u] += number of keys below mine[u], for a lane's first N entries.
  template <int N>
  __device__ void count_below(const uint64_t (&mine)[NE], int (&rk)[NE]) const {
#pragma unroll 4
    for (int j = 0; j < cnt; ++j) {
      const uint64_t o = key[j];
#pragma unroll
      for (int u = 0; u < (N < NE ? N : NE); ++u) rk[u] += o < mine[u];
    }
  }

  // The lane with entry e gets f(key, rank among the list's keys), which are
  // distinct.  All reads come before the first f.
  template <class F>
  __device__ void ranked(F&& f) {
    uint64_t mine[NE];
    int rk[NE];
    load(mine);
#pragma unroll
    for (int u = 0; u < NE; ++u) rk[u] = 0;
    // only the first entries of the lanes exist in a short list
    if (cnt <= 2 * GL)
      count_below<2>(mine, rk);
    else if (cnt <= 3 * GL)
      count_below<3>(mine, rk);
    else
      count_below<NE>(mine, rk);
    wave_sync();
    const int l = threadIdx.x % GL;
#pragma unroll
    for (int u = 0; u < NE; ++u)
      if (l + u * GL < cnt) f(mine[u], rk[u]);
  }

  static constexpr int LONG = 0;  // points of a span that is read as a whole (0: none)
  static __device__ uint64_t key_at(const float4& P, const float4& q) { return point_key(P, q); }

  __device__ void trim() {
    if (cnt < k) return;
    uint64_t mine[NE];
    load(mine);
    const int l = threadIdx.x % GL;
    unsigned d[NE], top = 0;
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      d[u] = (unsigned)(mine[u] >> 32);  // ~0 where there is no entry
      if (l + u * GL < cnt) top = max(top, d[u]);
    }
    // the smallest distance hi tried with at least k keys up to it
    unsigned lo = 0, hi = group_max<GL>(top);
    int have = cnt;
    while (have > k + SLACK && lo < hi) {
      const unsigned mid = lo + ((hi - lo) >> 1);
      int c = 0;
#pragma unroll
      for (int u = 0; u < NE; ++u) c += d[u] <= mid;
      c = group_sum<GL>(c);
      if (c >= k) {
        hi = mid;
        have = c;
      } else {
        lo = mid + 1;
      }
    }
    if (have > k + SLACK) {
      // more equal distances than fit: the k smallest keys by rank
      int rk[NE];
#pragma unroll
      for (int u = 0; u < NE; ++u) rk[u] = 0;
      count_below<NE>(mine, rk);
      wave_sync();
#pragma unroll
      for (int u = 0; u < NE; ++u)
        if (l + u * GL < cnt && rk[u] < k) key[rk[u]] = mine[u];
      wave_sync();
      cnt = k;
      bound = min(bound, key[k - 1]);
      return;
    }
    if (have < cnt) {
      cnt = 0;
#pragma unroll
      for (int u = 0; u < NE; ++u) push(mine[u], d[u] <= hi);
    }
    bound = min(bound, (uint64_t)(hi + 1) << 32);
  }

  // Appends the keys of the lanes that have one.
  __device__ void push(uint64_t w, bool pass) {
    const uint64_t m = __ballot(pass);
    if constexpr (GL == 16) {
      const int lane = threadIdx.x & 63;
      const unsigned mg = ((lane & 32 ? (unsigned)(m >> 32) : (unsigned)m) >> (lane & 16)) & 0xffffu;
      if (pass) key[cnt + __popc(mg & ((1u << (lane & 15)) - 1u))] = w;
      cnt += __popc(mg);
    } else {
      static_assert(GL == 64, "a group of 16 lanes or a wave");
      if (pass) key[cnt + __popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull))] = w;
      cnt += __popcll(m);
    }
  }
  // Number of keys below a bound.
  __device__ int count_under(uint64_t b) const {
    int c = 0;
    wave_sync();
    for (int e = threadIdx.x % GL; e < cnt; e += GL) c += key[e] < b;
    return group_sum<GL>(c);
  }
  // One candidate per lane (ok: this lane has one); room() comes before.
  __device__ void add(uint64_t w, bool ok) { push(w, ok && w < bound); }
  template <int U>
  __device__ void room() {
    if (cnt > CAP - U * GL) trim();
  }
  __device__ void settle() {}
  // The bound is about to be used again.
  __device__ void lower() { trim(); }
  // The keys are about to be met again.
  __device__ void again() {
    if (cnt >= k) {
      trim();
      ++bound;
    }
    cnt = 0;
  }
};

// Sum over the lanes before this one of its group (exclusive), and the
// group's total.
template <int GL>
__device__ inline int group_scan(int v, int& total) {
  int x = v;
  if constexpr (GL == 16) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row shift right by 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    total = __shfl(x, (int)(threadIdx.x & 63) | 15, 64);
  } else {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(x, off, 64);
      if (lane >= off) x += o;
    }
    total = __builtin_amdgcn_readlane(x, 63);
  }
  return x - v;
}

// Visits the points of the cells within radius R of the query's cell, but
// not those within radius inner (< 0: none), that can hold keys below the
// sink's bound.  A lane of the group looks up one row of cells at a time: the
// distance from the query to the row, the cells of it within the bound, and
// their span or, on both sides of the inner cube, two.  Spans are short (a
// dozen points), so they are cut into segments of 8 points, laid out in LDS
// (s_seg, GL * SEG_PER of them), and the group reads GL / 8 segments at once,
// U times before it uses the first.
//
// RU rows per lane are looked up at once (the two loads of a row are the
// longest wait of a search with many rows).  LARGE: of the cube only the rows
// inside the grid are enumerated.  Returns the number of points in
// the spans (of the group).
constexpr int SEG_PER = 4;

// The points of the lanes' long spans a, one span after the other, which are
// emptied: in a crowded cell (far outliers make the cells large) a segment of 8
// at a time costs more than its points.  30 000 points in one cell, nearest to
// 30 000 queries: 1.73 ms by segments, 0.6 so (1.05 by a search over all).
template <int GL, class Sink>
__device__ inline bool take_long(const GridJob& J, int2& a, const float4& q, Sink& L) {
  constexpr int U = Sink::LONG / GL;
  const int lane = threadIdx.x & 63, l = threadIdx.x % GL;
  bool any = false;
  for (;;) {
    const unsigned m = (unsigned)(__ballot(a.y - a.x >= Sink::LONG) >> (lane & 48)) & 0xffffu;
    static_assert(GL == 16, "a group's bits of the wave's");
    if (m == 0) return any;
    any = true;
    const int src = (lane & 48) + __builtin_ctz(m);
    const int x = __shfl(a.x, src, 64), y = __shfl(a.y, src, 64);
    for (int j = x; j < y; j += GL * U) {
      float4 P[U];
#pragma unroll
      for (int u = 0; u < U; ++u) P[u] = J.spts[min(j + u * GL + l, y - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u) L.add(Sink::key_at(P[u], q), true);  // (the last point again beyond the span)
    }
    if (lane == src) a = make_int2(0, 0);
  }
}

// The points of every lane's spans a and b; returns how many the lane's were.
template <int GL, int U, class Sink>
__device__ inline int take_spans(const GridJob& J, int2 a, int2 b, const float4& q, Sink& L, int2* s_seg) {
  const int l = threadIdx.x % GL;
  const int points = a.y - a.x + b.y - b.x;
  bool any = false;
  if constexpr (Sink::LONG > 0) {
    if (__any(points >= Sink::LONG)) {
      any = take_long<GL>(J, a, q, L);
      any |= take_long<GL>(J, b, q, L);
    }
  }
  int todo = ((a.y - a.x + 7) >> 3) + ((b.y - b.x + 7) >> 3);
  for (;;) {
    const int take = min(todo, SEG_PER);
    int total;
    const int at0 = group_scan<GL>(take, total);
    if (total == 0) break;
    any = true;
    wave_sync();
    for (int u = 0; u < take; ++u) {
      if (a.x >= a.y) {
        a = b;
        b = make_int2(0, 0);
      }
      s_seg[at0 + u] = make_int2(a.x, min(a.x + 8, a.y));
      a.x += 8;
    }
    todo -= take;
    wave_sync();
    for (int s = 0; s < total; s += U * (GL / 8)) {
      float4 P[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = s + u * (GL / 8) + (l >> 3);
        const int2 sg = e < total ? s_seg[e] : make_int2(0, 0);
        ok[u] = sg.x + (l & 7) < sg.y;
        P[u] = J.spts[ok[u] ? sg.x + (l & 7) : 0];
      }
      L.template room<U>();
#pragma unroll
      for (int u = 0; u < U; ++u) L.add(Sink::key_at(P[u], q), ok[u]);
      if constexpr (Sink::LONG == 0) L.settle();
    }
  }
  if (Sink::LONG > 0 && any) L.settle();
  return points;
}

template <int GL, int U, int RU, bool LARGE, class Sink>
__device__ inline int visit(const GridJob& J, const GridInfo& G, const Place& at, const float4& q, int R, int inner,
                            Sink& L, int2* s_seg) {
  const int l = threadIdx.x % GL;
  int ny = 2 * R + 1, nz = ny, y0 = -R, z0 = -R;
  if constexpr (LARGE) {
    y0 = slabs(at.c[1], G.dims[1], R, ny);
    z0 = slabs(at.c[2], G.dims[2], R, nz);
  }
  const int rows = ny * nz;
  const float inv_ny = 1.f / (float)ny;
  const float inv_h = (float)G.inv_h;
  int seen = 0;
  for (int r0 = 0; r0 < rows; r0 += GL * RU) {
    int2 a[RU], b[RU];
    const float reach2 = key_of(L.bound) * (inv_h * inv_h) * (1.f + 2e-5f);
#pragma unroll
    for (int v = 0; v < RU; ++v) {
      a[v] = b[v] = make_int2(0, 0);
      const int i = r0 + v * GL + l;
      int dz = (int)(((float)i + 0.5f) * inv_ny);
      int dy = i - dz * ny;
      if (dy < 0) dy += ny, --dz;
      if (dy >= ny) dy -= ny, ++dz;
      dz += z0;
      dy += y0;
      int xl, xr;
      if (i < rows && row_cells(G, at, R, dy, dz, reach2, xl, xr)) {
        const int cx = at.c[0];
        const int* st = J.starts + ((at.c[2] + dz) * G.dims[1] + at.c[1] + dy) * G.dims[0];
        if (max(abs(dy), abs(dz)) > inner) {
          a[v] = make_int2(st[xl], st[xr + 1]);
        } else {
          if (xl < cx - inner) a[v] = make_int2(st[xl], st[cx - inner]);
          if (xr > cx + inner) b[v] = make_int2(st[cx + inner + 1], st[xr + 1]);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < RU; ++v) seen += take_spans<GL, U>(J, a[v], b[v], q, L, s_seg);
  }
  return group_sum<GL>(seen);
}

// Every key below the sink's bound, by the listed blocks of cells: a wave
// measures 64 blocks at a time against the bound and visits those within it,
// a lane per row, the nearest block of all first.
template <int U, class Sink>
__device__ inline void visit_blocks(const GridJob& J, const GridInfo& G, const Place& at, const float4& q, Sink& L,
                                    int2* s_seg) {
  const int lane = threadIdx.x & 63;
  const float inv_h2 = (float)G.inv_h * (float)G.inv_h * (1.f + 2e-5f);
  auto gap_of = [&](int pb) {
    int bc[3];
    unpack_cell(G, pb, bc);
    return block_gap(at, bc);
  };
  auto visit_block = [&](int pb) {
    int bc[3];
    unpack_cell(G, pb, bc);
    int2 a = make_int2(0, 0);
    int cy, cz, xl, xr;
    if (block_row_cells(G, at, bc, lane, key_of(L.bound) * inv_h2, cy, cz, xl, xr)) {
      const int* st = J.starts + (cz * G.dims[1] + cy) * G.dims[0];
      a = make_int2(st[xl], st[xr + 1]);
    }
    take_spans<64, U>(J, a, make_int2(0, 0), q, L, s_seg);
  };
  const int nb = J.blocks[0];
  uint64_t best = ~0ull;
  for (int i = lane; i < nb; i += 64)
    best = min(best, (uint64_t)__float_as_uint(gap_of(J.blocks[1 + i])) << 32 | (unsigned)i);
  for (int off = 32; off > 0; off >>= 1) best = min(best, (uint64_t)__shfl_xor((unsigned long long)best, off, 64));
  const int first = nb > 0 ? (int)(unsigned)best : -1;
  if (first < 0) return;
  visit_block(__builtin_amdgcn_readfirstlane(J.blocks[1 + first]));
  L.lower();
  for (int i0 = 0; i0 < nb; i0 += 64) {
    const int i = i0 + lane;
    const int pb = J.blocks[1 + min(i, nb - 1)];
    const float g2 = gap_of(pb);
    bool want = i < nb && i != first;
    for (;;) {
      const uint64_t m = __ballot(want && !(g2 > key_of(L.bound) * inv_h2));
      if (m == 0) break;
      const int j = __builtin_ctzll(m);
      if (lane == j) want = false;
      visit_block(__builtin_amdgcn_readlane(pb, j));
      L.lower();
    }
  }
}

constexpr int KF_ROWS = 4;
// Every key below the sink's bound: a wave looks at the cells within 3, 8 and
// 18 of the query's.  If the bound then still reaches further, the cells in
// reach are mostly empty (in a cloud that is mostly surfaces) and the listed
// blocks tell where the points are.  The sink's again() forgets the keys but
// not the bound.
template <int U, int RMAX, class Sink>
__device__ inline void visit_reach(const GridJob& J, const GridInfo& G, const Place& at, const float4& q, Sink& L,
                                   int2* s_seg) {
  const int rmax = max(G.dims[0], max(G.dims[1], G.dims[2]));
  for (int inner = -1, R = 3; R <= RMAX; R = 2 * R + 2) {
    R = min(R, cells_reached(G, at, L.bound, rmax));
    if (R <= inner) return;
    visit<64, U, KF_ROWS, false>(J, G, at, q, R, inner, L, s_seg);
    L.lower();
    inner = R;
  }
  if (cells_reached(G, at, L.bound, rmax) <= RMAX) return;
  L.again();
  visit_blocks<U>(J, G, at, q, L, s_seg);
}

constexpr int KN_BT = 256;
constexpr int KN_G = 16;                // lanes per query
constexpr int KN_U = 3;
constexpr int KN_CAP = 128;             // list entries: cut above 80, eight per lane
constexpr int KN_STRIDE = KN_CAP + 2;   // the groups' lists start in different LDS banks
constexpr int KN_Q = KN_BT / KN_G;      // queries of a block at a time
using QueryList = KeyList<KN_G, KN_CAP>;

// Writes a settled query's list: the k smallest keys in order, -1 where fewer
// finite points than k exist.
template <int GL, class List>
__device__ inline void write_list(List& L, int k, int32_t* __restrict__ out) {
  L.ranked([&](uint64_t w, int r) {
    if (r < k) out[r] = (int32_t)(uint32_t)w;
  });
  for (int e = L.cnt + (int)(threadIdx.x % GL); e < k; e += GL) out[e] = -1;
}

// Lists of the queries knn_kernel leaves, counts first: near[0].x of the
// queries with k points in their 27 cells, near[0].y of the others, which are
// listed from the end of the same array (size entries).
__device__ inline void leave_query(int2* list, int size, int cloud, int t, bool near) {
  if (near)
    list[1 + atomicAdd(&list[0].x, 1)] = make_int2(cloud, t);
  else
    list[size - atomicAdd(&list[0].y, 1)] = make_int2(cloud, t);
}

// Queries [block rounds KN_Q, ...) of a cloud in cell order, KN_Q at a time.
__global__ __launch_bounds__(KN_BT, 4) void knn_kernel(GridArgs A, int k, int rounds, int2* __restrict__ far,
                                                       int far_size) {
  __shared__ uint64_t s_key[KN_Q * KN_STRIDE];
  __shared__ int2 s_seg[KN_Q][KN_G * SEG_PER];
  int block, cloud;
  const GridJob J = job_of(A, block, &cloud);
  const GridInfo G = block_grid(J.gi);
  const int grp = threadIdx.x / KN_G, l = threadIdx.x % KN_G;
  for (int round = 0; round < rounds; ++round) {
    const int t = (block * rounds + round) * KN_Q + grp;
    if (t >= J.n) return;  // no block barrier below; a group leaves as a whole
    const float4 q = J.spts[t];
    int32_t* out = J.nbr + (int64_t)__float_as_int(q.w) * k;
    // a query with a non-finite coordinate has no finite key to any point:
    // its list is empty (and searching for one would visit every cell)
    if (!(isfinite(q.x) && isfinite(q.y) && isfinite(q.z))) {
      for (int e = l; e < k; e += KN_G) out[e] = -1;
      continue;
    }
    Place at;
    unpack_cell(G, J.scell[t], at.c);
    at.set(G, q);
    const int own = cell_index(G, at.c);
    const bool dense = J.starts[own + 1] - J.starts[own] >= k;
    const uint64_t edge = cube_bound(G, at, 1);
    // the 27 cells, for keys below the edge; a dense query's own cell first,
    // for any keys, whose k-th limits the rest
    QueryList L{s_key + grp * KN_STRIDE, 0, k, dense ? KEY_INF : edge};
    int seen = visit<KN_G, KN_U, 1, false>(J, G, at, q, dense ? 0 : 1, -1, L, s_seg[grp]);
    if (dense) {
      L.trim();
      L.bound = min(L.bound, edge);
      seen += visit<KN_G, KN_U, 1, false>(J, G, at, q, 1, 0, L, s_seg[grp]);
    }
    // keys of a dense query's own cell may lie beyond the edge
    bool found = edge == KEY_INF || (dense ? L.count_under(edge) : L.cnt) >= k;
    if (found) {
      if (L.cnt > 3 * KN_G) L.trim();
      write_list<KN_G>(L, k, out);
    } else if (l == 0) {
      leave_query(far, far_size, cloud, t, seen >= k);
    }
  }
}

constexpr int KF_CAP = 256;    // list entries of a wave: cut above 128, four per lane
constexpr int KF_U = 2;

// The queries knn_kernel left.  Those with k points in their 27 cells, 16
// lanes each: their k-th key lies a little beyond the bound of these cells, so
// the bound is raised until k keys are below it (searching for any keys
// first would fill the list from the dense cells next to a sparse place).  The
// others, a wave each: the k-th key of the 128 points around the query in the
// sorted array (its own and the next rows of cells) bounds a search by blocks
// of cells.  Waves take the second kind first, the longer ones.
__global__ __launch_bounds__(KN_BT) void knn_far_kernel(GridArgs A, int k, const int2* __restrict__ far,
                                                        int far_size) {
  __shared__ union {
    struct {
      uint64_t key[(KN_BT / 64) * KF_CAP];
      int2 seg[KN_BT / 64][64 * SEG_PER];
    } w;
    struct {
      uint64_t key[KN_Q * KN_STRIDE];
      int2 seg[KN_Q][KN_G * SEG_PER];
    } g;
  } sh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int waves = (gridDim.x * KN_BT) >> 6, first_wave = (blockIdx.x * KN_BT + threadIdx.x) >> 6;
  const int n_near = far[0].x, n_far = far[0].y;
  for (int f = first_wave; f < n_far; f += waves) {
    const int2 ct = far[far_size - f];
    const GridJob J = job_at(A, ct.x);
    const GridInfo G = *J.gi;
    const float4 q = J.spts[ct.y];
    Place at;
    unpack_cell(G, J.scell[ct.y], at.c);
    at.set(G, q);
    KeyList<64, KF_CAP> L{sh.w.key + wave * KF_CAP, 0, k, KEY_INF};
    {
      const int first = max(0, min(ct.y - 64, J.n - 128));
      const float4 P0 = J.spts[min(first + lane, J.n - 1)], P1 = J.spts[min(first + 64 + lane, J.n - 1)];
      L.add(point_key(P0, q), first + lane < J.n);
      L.add(point_key(P1, q), first + 64 + lane < J.n);
      L.again();
    }
    visit_reach<KF_U, 18>(J, G, at, q, L, sh.w.seg[wave]);
    if (L.cnt > 3 * 64) L.trim();
    write_list<64>(L, k, J.nbr + (int64_t)__float_as_int(q.w) * k);
  }
  __syncthreads();  // the lists of the other kind lie in the same LDS
  const int grp = threadIdx.x / KN_G;
  for (int f = blockIdx.x * KN_Q + grp; f < n_near; f += gridDim.x * KN_Q) {
    const int2 ct = far[1 + f];
    const GridJob J = job_at(A, ct.x);
    const GridInfo G = *J.gi;
    const float4 q = J.spts[ct.y];
    Place at;
    unpack_cell(G, J.scell[ct.y], at.c);
    at.set(G, q);
    const int rmax = max(G.dims[0], max(G.dims[1], G.dims[2]));
    // fewer than k keys below the cube's bound: all keys below twice that
    // distance squared, then five times, ...
    QueryList L{sh.g.key + grp * KN_STRIDE, 0, k, 0};
    for (float reach2 = widen_first(cube_bound(G, at, 1));; reach2 *= WIDEN) {
      bool last;
      L.cnt = 0;
      const int R = widen(G, at, reach2, rmax, L.bound, last);
      visit<KN_G, KN_U, 2, true>(J, G, at, q, R, -1, L, sh.g.seg[grp]);
      if (L.cnt >= k || last) break;
    }
    write_list<KN_G>(L, k, J.nbr + (int64_t)__float_as_int(q.w) * k);
  }
}

// Curvature from the neighbour lists (FP64 covariance, 1/k, centred), one
// block of CURV_BT points.  A point's list is k consecutive indices, so with
// one point per thread every load instruction of a wave would touch 64
// different rows; the block's rows (contiguous in memory) are therefore
// copied into LDS with coalesced loads first, at an odd row stride so that
// the threads' reads of their own rows meet no bank conflict.  The
// neighbours' packed coordinates (p4) are then read in groups of CURV_G, each
// group's loads all requested before the first is used, in one pass: the
// sums are taken of the offsets from the list's first point (the query
// itself unless duplicates come first), C = S2 / k - (S1 / k)(S1 / k)^T,
// which is the centred covariance for any shift and, with a shift inside the
// neighbourhood, keeps the FP64 cancellation at the rounding of the offsets.
constexpr int CURV_BT = 256;
constexpr int CURV_G = 8;

__device__ inline int curv_stride(int k) { return k | 1; }

// Points [b CURV_BT, min(n, (b + 1) CURV_BT)); lds holds CURV_BT rows of
// curv_stride(k) ints.  Every thread reaches the barrier.
__device__ inline void curvature_block(const float4* __restrict__ p4, int n, int k, const int32_t* __restrict__ idx,
                                       float* __restrict__ a_out, int b, int* lds) {
  const int p0 = b * CURV_BT;
  const int cnt = min(CURV_BT, n - p0);
  const int st = curv_stride(k);
  {
    // element e = threadIdx.x + CURV_BT i of the block's cnt k indices is
    // column c of row r; (r, c) advance by (CURV_BT / k, CURV_BT % k)
    const int32_t* src = idx + (int64_t)p0 * k;
    const int dr = CURV_BT / k, dc = CURV_BT % k;
    int r = threadIdx.x / k, c = threadIdx.x % k;
#pragma unroll 4
    for (int e = threadIdx.x; e < cnt * k; e += CURV_BT) {
      lds[r * st + c] = src[e];
      r += dr;
      c += dc;
      if (c >= k) {
        c -= k;
        ++r;
      }
    }
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t >= cnt) return;
  const int q = p0 + t;
  const int* nb = lds + t * st;
  bool missing = false;
  double sh[3] = {0, 0, 0}, S1[3] = {0, 0, 0}, S2[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll 1
  for (int s0 = 0; s0 < k; s0 += CURV_G) {
    int id[CURV_G];
#pragma unroll
    for (int u = 0; u < CURV_G; ++u) id[u] = s0 + u < k ? nb[s0 + u] : 0;
    float4 P[CURV_G];
#pragma unroll
    for (int u = 0; u < CURV_G; ++u) P[u] = p4[max(id[u], 0)];
    if (s0 == 0) {
      sh[0] = (double)P[0].x;
      sh[1] = (double)P[0].y;
      sh[2] = (double)P[0].z;
    }
#pragma unroll
    for (int u = 0; u < CURV_G; ++u) {
      if (s0 + u < k) {
        missing |= id[u] < 0;
        const double dx = (double)P[u].x - sh[0], dy = (double)P[u].y - sh[1], dz = (double)P[u].z - sh[2];
        S1[0] += dx;
        S1[1] += dy;
        S1[2] += dz;
        S2[0] += dx * dx;
        S2[1] += dy * dy;
        S2[2] += dz * dz;
        S2[3] += dx * dy;
        S2[4] += dx * dz;
        S2[5] += dy * dz;
      }
    }
  }
  if (missing) {
    a_out[q] = NAN;
    return;
  }
  const double invk = 1.0 / (double)k;
  const double mx = S1[0] * invk, my = S1[1] * invk, mz = S1[2] * invk;
  const double C[6] = {S2[0] * invk - mx * mx, S2[1] * invk - my * my, S2[2] * invk - mz * mz,
                       S2[3] * invk - mx * my, S2[4] * invk - mx * mz, S2[5] * invk - my * mz};
  double lam[3];
  eig_psd3(C, lam);
  const double tr = C[0] + C[1] + C[2];
  a_out[q] = (tr > 0.0) ? (float)(lam[2] / tr) : 0.f;
}

// Dynamic LDS of the curvature kernels: CURV_BT rows of curv_stride(k) ints.
inline size_t curv_lds_bytes(int k) { return sizeof(int) * (size_t)CURV_BT * (size_t)(k | 1); }

__global__ __launch_bounds__(CURV_BT) void curvature_kernel(GridArgs A, int k) {
  extern __shared__ int s_nb[];
  int b;
  const GridJob J = job_of(A, b);
  if (J.a_out) curvature_block(J.p4, J.n, k, J.nbr, J.a_out, b, s_nb);
}

// ------------------------------------------------------------------- host
// Clouds of up to SMALL_N points (in a batch SMALL_BATCH_N, where the clouds
// are built side by side) are built by one block, which takes 11 us at 1 024
// points, 27 at 8 192 and 47 at 16 384; the six launches of the large build
// take 32 us at 16 385 and 35 at 36 000, and the gaps between them.
constexpr int SMALL_N = 8192;
constexpr int SMALL_BATCH_N = 65535;  // 16-bit cell starts

static int large_cells(int n) {
  int m = 1024;
  while (m < 4 * n && m < (1 << 24)) m <<= 1;
  return m;
}
static int small_cells(int n) { return std::min(2 * SM_WORDS, std::max(1024, 4 * n)); }

namespace {

size_t up256(size_t b) { return (b + 255) & ~size_t(255); }

// Workspace of one cloud, carved at ws (nullptr: size only).
size_t carve_job(char* ws, int n, int k, GridJob* J) {
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* r = ws + o;
    o += up256(bytes);
    return (void*)r;
  };
  const int mc = large_cells(n);  // never below small_cells of the sizes that use them
  const int cells = std::max(mc, small_cells(n));
  GridJob T{};
  T.gi = (GridInfo*)take(sizeof(GridInfo));
  T.cell_of = (int*)take(sizeof(int) * (size_t)n);
  T.rank = (int*)take(sizeof(int) * (size_t)n);
  T.counts = (int*)take(sizeof(int) * (size_t)cells);
  T.starts = (int*)take(sizeof(int) * ((size_t)cells + 1));
  T.part = (int*)take(sizeof(int) * ((size_t)LG_PART + cells / LG_SCAN + 1));
  T.spts = (float4*)take(sizeof(float4) * (size_t)n);
  T.scell = (int*)take(sizeof(int) * (size_t)n);
  T.p4 = (float4*)take(sizeof(float4) * (size_t)n);
  T.nbr = (int32_t*)take(sizeof(int32_t) * (size_t)n * k);
  T.blocks = (int*)take(sizeof(int) * ((size_t)n + 1));
  if (J) {
    T.n = n;
    *J = T;
  }
  return o;
}

size_t far_bytes(int64_t points) { return up256(sizeof(int2) * (size_t)(points + 2)); }

hipError_t build_large(const GridJob& J, int2* far, hipStream_t st) {
  const dim3 blocks(LG_BLOCKS), bt(LG_BT);
  const unsigned ns = (unsigned)((J.max_cells + LG_SCAN - 1) / LG_SCAN);
  hipLaunchKernelGGL(grid_box_kernel, blocks, bt, 0, st, J, far);
  hipLaunchKernelGGL(grid_occupancy_kernel, blocks, bt, 0, st, J);
  hipLaunchKernelGGL(grid_count_kernel, dim3((unsigned)std::min(2048, (J.n + LG_BT - 1) / LG_BT)), bt, 0, st, J);
  hipLaunchKernelGGL(grid_sums_kernel, dim3(ns), dim3(1024), 0, st, J);
  hipLaunchKernelGGL(grid_starts_kernel, dim3(ns), dim3(1024), 0, st, J);
  const int pb = (J.n + LG_BT - 1) / LG_BT;
  hipLaunchKernelGGL(grid_scatter_kernel, dim3((unsigned)(pb + std::min(256, pb))), bt, 0, st, J, pb);
  return hipGetLastError();
}

hipError_t build_one(GridJob& J, int2* far, hipStream_t st) {
  if (J.n > SMALL_N) {
    J.max_cells = large_cells(J.n);
    return build_large(J, far, st);
  }
  J.max_cells = small_cells(J.n);
  hipLaunchKernelGGL(grid_small_kernel, dim3(1), dim3(SM_BT), sizeof(int) * (size_t)((J.max_cells + 1) / 2), st,
                     GridArgs{J, nullptr, nullptr}, far);
  return hipGetLastError();
}

}  // namespace

size_t grid_knn_workspace(int n, int k) { return carve_job(nullptr, n, k, nullptr) + far_bytes(n); }

hipError_t launch_grid_knn(const float* x, const float* y, const float* z, int n, int k, float* a_out,
                           int32_t* idx_out, void* ws, hipStream_t st) {
  GridJob J;
  int2* far = (int2*)((char*)ws + carve_job((char*)ws, n, k, &J));
  J.x = x, J.y = y, J.z = z, J.a_out = a_out;
  J.occ = grid_occ(k);
  if (idx_out) J.nbr = idx_out;
  if (hipError_t e = build_one(J, far, st)) return e;
  const GridArgs A{J, nullptr, nullptr};
  // a few queries per group where there are many: fewer block starts
  const int rounds = n <= 65536 ? 1 : 4;
  hipLaunchKernelGGL(knn_kernel, dim3((unsigned)((n + KN_Q * rounds - 1) / (KN_Q * rounds))), dim3(KN_BT), 0, st, A, k,
                     rounds, far, n + 1);
  hipLaunchKernelGGL(knn_far_kernel, dim3(512), dim3(KN_BT), 0, st, A, k, far, n + 1);
  if (a_out)
    hipLaunchKernelGGL(curvature_kernel, dim3((unsigned)((n + CURV_BT - 1) / CURV_BT)), dim3(CURV_BT),
                       curv_lds_bytes(k), st, A, k);
  return hipGetLastError();
}

size_t grid_knn_batch_workspace(const int* n, int n_clouds, int k) {
  size_t b = 0;
  int64_t blocks = 0, points = 0;
  for (int c = 0; c < n_clouds; ++c) {
    b += carve_job(nullptr, n[c], k, nullptr);
    blocks += (n[c] + 255) / 256;
    points += n[c];
  }
  return b + up256(sizeof(GridJob) * (size_t)n_clouds) + up256(sizeof(int2) * (size_t)(blocks + n_clouds)) +
         far_bytes(points);
}

// Many clouds: one launch per phase for all of them, through a table of jobs
// and a list of (cloud, block of 256 points).  Clouds above SMALL_BATCH_N
// points build their grids one after the other.
hipError_t launch_grid_knn_batch(const float* const* x, const float* const* y, const float* const* z, const int* n,
                                 float* const* a_out, int32_t* const* idx_out, int n_clouds, int k, void* ws,
                                 hipStream_t st) {
  if (n_clouds < 1) return hipSuccess;
  // one host table, one copy: the jobs, the (cloud, 0) list of the small
  // builds, the (cloud, block) list
  const size_t jobs_bytes = up256(sizeof(GridJob) * (size_t)n_clouds);
  std::vector<GridJob> jobs(n_clouds);
  std::vector<int2> small, bmap;
  char* p = (char*)ws;
  int64_t points = 0;
  int cells = 0;
  for (int c = 0; c < n_clouds; ++c) {
    GridJob& J = jobs[c];
    p += carve_job(p, n[c], k, &J);
    J.x = x[c], J.y = y[c], J.z = z[c], J.a_out = a_out ? a_out[c] : nullptr;
    J.occ = grid_occ(k);
    if (idx_out && idx_out[c]) J.nbr = idx_out[c];
    if (n[c] <= SMALL_BATCH_N) {
      J.max_cells = small_cells(n[c]);
      cells = std::max(cells, J.max_cells);
      small.push_back(make_int2(c, 0));
    } else {
      J.max_cells = large_cells(n[c]);
    }
    for (int b = 0; b < (n[c] + 255) / 256; ++b) bmap.push_back(make_int2(c, b));
    points += n[c];
  }
  // the largest first: a build takes as long as its cloud is large
  std::stable_sort(small.begin(), small.end(), [&](const int2& a, const int2& b) { return n[a.x] > n[b.x]; });
  std::vector<char> table(jobs_bytes + sizeof(int2) * (small.size() + bmap.size()));
  std::copy((const char*)jobs.data(), (const char*)(jobs.data() + n_clouds), table.data());
  std::copy((const char*)small.data(), (const char*)(small.data() + small.size()), table.data() + jobs_bytes);
  std::copy((const char*)bmap.data(), (const char*)(bmap.data() + bmap.size()),
            table.data() + jobs_bytes + sizeof(int2) * small.size());
  const GridJob* d_jobs = (const GridJob*)p;
  const int2* d_small = (const int2*)(p + jobs_bytes);
  const int2* d_bmap = d_small + small.size();
  int2* far = (int2*)(p + jobs_bytes + up256(sizeof(int2) * (small.size() + bmap.size())));
  hipError_t e = hipMemcpyAsync(p, table.data(), table.size(), hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return e;
  // the copy reads a host vector that goes out of scope below
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return e;
  for (int c = 0; c < n_clouds; ++c)
    if (n[c] > SMALL_BATCH_N)
      if ((e = build_large(jobs[c], far, st)) != hipSuccess) return e;
  // (the far count is cleared by every large build and by cloud 0's small
  // one; all of them run before the search)
  if (!small.empty())
    hipLaunchKernelGGL(grid_small_kernel, dim3((unsigned)small.size()), dim3(SM_BT), sizeof(int) * (size_t)((cells + 1) / 2), st,
                       GridArgs{GridJob{}, d_jobs, d_small}, far);
  const GridArgs A{GridJob{}, d_jobs, d_bmap};
  const dim3 gb((unsigned)bmap.size());
  hipLaunchKernelGGL(knn_kernel, gb, dim3(KN_BT), 0, st, A, k, 256 / KN_Q, far, (int)points + 1);
  hipLaunchKernelGGL(knn_far_kernel, dim3(1024), dim3(KN_BT), 0, st, A, k, far, (int)points + 1);
  hipLaunchKernelGGL(curvature_kernel, gb, dim3(CURV_BT), curv_lds_bytes(k), st, A, k);
  return hipGetLastError();
}

// ---------------------------------------------------------------- nearest
// The nearest point kept by a group of GL lanes: each lane's own best key,
// and the group's after every batch, which bounds the cells still visited.
template <int GL, bool FUSED>
struct Nearest {
  uint64_t best, bound;

  static constexpr int LONG = GL == 16 ? 32 : 0;  // (the same point twice does no harm)
  static __device__ uint64_t key_at(const float4& P, const float4& q) {
    return FUSED ? point_key_fused(P, q) : point_key(P, q);
  }

  __device__ void add(uint64_t w, bool ok) {
    if (ok && w < best) best = w;
  }
  template <int U>
  __device__ void room() {}
  __device__ void lower() {}
  __device__ void again() {}
  __device__ void settle() {
    if constexpr (GL == 64) {
      best = min(best, other<32>());
      best = min(best, other<16>());
    }
    best = min(best, other<8>());
    best = min(best, other<4>());
    best = min(best, other<2>());
    best = min(best, other<1>());
    bound = min(bound, best);
  }
  template <int OFF>
  __device__ uint64_t other() const {
    return (uint64_t)xor_lane_u<OFF>((unsigned)(best >> 32)) << 32 | xor_lane_u<OFF>((unsigned)best);
  }
};

constexpr int NN_RMAX = 3;  // cells from its own a group searches for a query before a wave takes it

// Nearest point of the grid's cloud to each query (any points, inside or
// outside the grid's box) among the points whose key is <= max_key: the same
// (key, index) order as the neighbour lists, 16 lanes per query.  A query with
// no such point, or with a non-finite coordinate, gets index -1 and key +inf.
// Queries not settled within NN_RMAX cells go to the far list.  Bound by the
// latency of the dependent loads (start of a row, its points): 96 us for
// 250 000 queries near 307 200 points, where a lane per query took 872 us.
template <bool FUSED>
__global__ __launch_bounds__(KN_BT, 7) void nearest_kernel(GridJob J, const float* __restrict__ qx,
                                                        const float* __restrict__ qy, const float* __restrict__ qz,
                                                        int nq, float max_key, int32_t* __restrict__ nn,
                                                        float* __restrict__ key, int2* __restrict__ far) {
  __shared__ int2 s_seg[KN_Q][KN_G * SEG_PER];
  const GridInfo G = block_grid(J.gi);
  const int grp = threadIdx.x / KN_G, l = threadIdx.x % KN_G;
  const int t = blockIdx.x * KN_Q + grp;
  if (t >= nq) return;  // no block barrier below; a group leaves as a whole
  const float4 q = make_float4(qx[t], qy[t], qz[t], 0.f);
  Nearest<KN_G, FUSED> N{KEY_INF, ((uint64_t)__float_as_uint(max_key) << 32) | 0xffffffffu};
  bool found = true;
  if (isfinite(q.x) && isfinite(q.y) && isfinite(q.z)) {
    Place at;
    cell_of_point(G, q.x, q.y, q.z, at.c);
    at.set(G, q);
    // the query's own cell first: in a dense cloud its best key leaves little
    // of the others
    for (int inner = -1, R = 0;;) {
      visit<KN_G, KN_U, 1, false>(J, G, at, q, R, inner, N, s_seg[grp]);
      const int want = cells_reached(G, at, N.bound, 1 << 20);
      found = want <= R || cube_bound(G, at, R) == KEY_INF;
      if (found || (R > 0 && want > NN_RMAX)) break;
      inner = R;
      R = R == 0 ? 1 : want;
    }
  }
  if (l != 0) return;
  if (!found) {
    far[1 + atomicAdd(&far[0].x, 1)] = make_int2(0, t);
    return;
  }
  const bool hit = N.best < KEY_INF && key_of(N.best) <= max_key;
  nn[t] = hit ? (int32_t)(uint32_t)N.best : -1;
  key[t] = hit ? key_of(N.best) : INFINITY;
}

// The queries nearest_kernel left, one wave each: 64 points around the place
// in the sorted array where the query's cell begins give a first bound for a
// search of the cells within reach or, if these are many, by blocks of cells.
// Five waves per SIMD: with four, 3.45 instead of 3.31 ms for 250 000 queries off
// a surface of 307 200 points.
constexpr int NF_RMAX = 6;

template <bool FUSED>
__global__ __launch_bounds__(KN_BT, 5) void nearest_far_kernel(GridJob J, const float* __restrict__ qx,
                                                            const float* __restrict__ qy,
                                                            const float* __restrict__ qz, float max_key,
                                                            int32_t* __restrict__ nn, float* __restrict__ key,
                                                            const int2* __restrict__ far) {
  __shared__ int2 s_seg[KN_BT / 64][64 * SEG_PER];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int total = far[0].x;
  const GridInfo G = block_grid(J.gi);
  for (int f = (blockIdx.x * KN_BT + threadIdx.x) >> 6; f < total; f += (gridDim.x * KN_BT) >> 6) {
    const int t = far[1 + f].y;
    const float4 q = make_float4(qx[t], qy[t], qz[t], 0.f);
    Place at;
    cell_of_point(G, q.x, q.y, q.z, at.c);
    at.set(G, q);
    at.set_above(G, q);
    Nearest<64, FUSED> N{KEY_INF, ((uint64_t)__float_as_uint(max_key) << 32) | 0xffffffffu};
    const int first = max(0, min(J.starts[cell_index(G, at.c)] - 32, J.n - 64));
    N.add(N.key_at(J.spts[min(first + lane, J.n - 1)], q), true);
    N.settle();
    if (cells_reached(G, at, N.bound, 1 << 20) <= NF_RMAX)
      visit<64, KF_U, 1, false>(J, G, at, q, NF_RMAX, -1, N, s_seg[wave]);
    else
      visit_blocks<KF_U>(J, G, at, q, N, s_seg[wave]);
    if (lane == 0) {
      const bool hit = N.best < KEY_INF && key_of(N.best) <= max_key;
      nn[t] = hit ? (int32_t)(uint32_t)N.best : -1;
      key[t] = hit ? key_of(N.best) : INFINITY;
    }
  }
}

// Workspace: the grid's, and a far list of nq entries.
size_t grid_nn_workspace(int n, int nq) { return carve_job(nullptr, n, 1, nullptr) + far_bytes(nq); }

hipError_t launch_grid_nn(const float* x, const float* y, const float* z, int n, const float* qx, const float* qy,
                          const float* qz, int nq, float max_key, bool fused, int32_t* nn, float* key, void* ws,
                          hipStream_t st) {
  GridJob J;
  int2* far = (int2*)((char*)ws + carve_job((char*)ws, n, 1, &J));
  J.x = x, J.y = y, J.z = z;
  J.occ = 4.0f;
  J.reach = std::min(1e30f, 1.002f * std::sqrt(max_key));
  if (hipError_t e = build_one(J, far, st)) return e;
  auto search = fused ? nearest_kernel<true> : nearest_kernel<false>;
  auto search_far = fused ? nearest_far_kernel<true> : nearest_far_kernel<false>;
  hipLaunchKernelGGL(search, dim3((unsigned)((nq + KN_Q - 1) / KN_Q)), dim3(KN_BT), 0, st, J, qx, qy, qz, nq, max_key,
                     nn, key, far);
  hipLaunchKernelGGL(search_far, dim3(2048), dim3(KN_BT), 0, st, J, qx, qy, qz, max_key, nn, key, far);
  return hipGetLastError();
}

}  // namespace sgr

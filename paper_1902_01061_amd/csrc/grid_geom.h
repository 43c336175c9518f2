// Geometry of the neighbour search's uniform grid: its cells, and the lower
// bounds by which a search leaves cells out.  Host-callable, so that a serial
// search with the same bounds can be checked against brute force on the CPU.
#pragma once
#include "common.h"

namespace sgr {

struct GridInfo {
  float lo[3];
  float h;
  double inv_h;
  int dims[3];
  int ncells;
  int sh[2];      // where the second and third coordinate of a packed cell begin
  double ext[3];  // bounding-box extents (for re-sizing the cells)
};

// Cell counts per axis for cell size h, grown by 10 % steps until the grid
// has at most max_cells (up to 2^24) cells: a long cloud may have nearly all of
// them along one axis.  No cell is so small that its square, or a key of that
// size, underflows in FP32.
SGR_HD void grid_dims(GridInfo& G, double h, int max_cells) {
  int d[3];
  h = fmax(h, 1e-18);
  for (int it = 0; it < 400; ++it) {
    const double ih = 1.0 / h;
    double tot = 1.0;
    for (int a = 0; a < 3; ++a) {
      const double c = fmin(16777216.0, floor(G.ext[a] * ih) + 1.0);
      d[a] = (int)c;
      tot *= c;
    }
    if (tot <= (double)max_cells) break;
    h *= 1.1;
  }
  G.h = (float)h;
  G.inv_h = 1.0 / (double)G.h;
  for (int a = 0; a < 3; ++a) G.dims[a] = d[a];
  G.ncells = d[0] * d[1] * d[2];
  G.sh[0] = d[0] > 1 ? 32 - __builtin_clz(d[0] - 1) : 0;
  G.sh[1] = G.sh[0] + (d[1] > 1 ? 32 - __builtin_clz(d[1] - 1) : 0);
}

// Trial grid from the box of the finite points (lo > hi: none): about two
// points per cell of the bounding volume; flat or linear clouds fall back to
// their non-degenerate extents.
SGR_HD GridInfo grid_trial(const float box[6], int n, int max_cells) {
  GridInfo G;
  double e[3];
  for (int a = 0; a < 3; ++a) {
    const bool any = box[a] <= box[3 + a];  // some finite point
    G.lo[a] = any ? box[a] : 0.f;
    e[a] = any ? (double)box[3 + a] - (double)box[a] : 0.0;
    G.ext[a] = e[a];
  }
  const double hi = fmax(e[0], fmax(e[1], e[2])), lo = fmin(e[0], fmin(e[1], e[2]));
  const double mid = fmax(fmin(e[0], e[1]), fmin(fmax(e[0], e[1]), e[2]));
  const double rho = 2.0;
  double h;
  if (lo > 1e-6 * hi)
    h = cbrt(hi * mid * lo * rho / n);
  else if (mid > 1e-6 * hi)
    h = sqrt(hi * mid * rho / n);
  else
    h = hi * rho / n;
  if (!(h > 0 && h < INFINITY)) h = 1.0;
  grid_dims(G, h, max_cells);
  return G;
}

// Final cell size from the trial grid's occupancy mu, the mean over the
// points of their cell's count.  Scans are surfaces, whose counts go with the
// side squared; a cloud with fewer points per cell than wanted is taken as a
// volume.
// A search for points within `reach` settles every query in its 27 cells
// when they are that large.
SGR_HD void grid_resize(GridInfo& G, double mu, float occ, float reach, int max_cells) {
  const double f = (double)occ / mu;
  grid_dims(G, (double)G.h * (f < 1.0 ? sqrt(f) : cbrt(f)), max_cells);
  if (G.h < reach && reach <= 2.f * G.h) grid_dims(G, (double)reach, max_cells);
}

// Cell coordinates and cell faces are computed in FP64 so that rounding
// cannot move a point across a face by more than a negligible fraction of a
// cell, whatever the offset of the cloud from the origin.  The last cell of an
// axis holds every point beyond it: with many cells, whose size is rounded to
// FP32, the points may reach a little further.
SGR_HD int cell_coord(float p, float lo, double inv_h, int dim) {
  const double u = floor(((double)p - (double)lo) * inv_h);
  return u < 0.0 ? 0 : (u >= (double)dim ? dim - 1 : (int)u);
}

SGR_HD int cell_index(const GridInfo& G, const int c[3]) {
  return (c[2] * G.dims[1] + c[1]) * G.dims[0] + c[0];
}
SGR_HD void cell_of_point(const GridInfo& G, float x, float y, float z, int c[3]) {
  c[0] = cell_coord(x, G.lo[0], G.inv_h, G.dims[0]);
  c[1] = cell_coord(y, G.lo[1], G.inv_h, G.dims[1]);
  c[2] = cell_coord(z, G.lo[2], G.inv_h, G.dims[2]);
}
SGR_HD int cell_index(const GridInfo& G, float x, float y, float z) {
  int c[3];
  cell_of_point(G, x, y, z, c);
  return cell_index(G, c);
}
// A cell's coordinates (or a block of cells') in one word of at most 27 bits.
SGR_HD int pack_cell(const GridInfo& G, const int c[3]) { return c[0] | c[1] << G.sh[0] | c[2] << G.sh[1]; }
SGR_HD void unpack_cell(const GridInfo& G, int p, int c[3]) {
  c[0] = p & ((1 << G.sh[0]) - 1);
  c[1] = (p & ((1 << G.sh[1]) - 1)) >> G.sh[0];
  c[2] = p >> G.sh[1];
}

SGR_HDI int min2(int a, int b) { return a < b ? a : b; }
SGR_HDI int max2(int a, int b) { return a > b ? a : b; }

SGR_HD float key_of(uint64_t w) { return __builtin_bit_cast(float, (uint32_t)(w >> 32)); }
constexpr uint64_t KEY_INF = 0x7f800000ull << 32;  // no key of a finite distance reaches it

// A query's place in the grid: its cell and its position in it in cell units,
// formed in FP64 (in [0, 1) inside the grid, from 0 up in the last cell; beyond
// it for a query outside, whose cell is the nearest).  Distances in cell units
// below are floats with a margin of 1e-3 of a cell, which covers their rounding
// and that of the cells, and 2e-5 relative for the float32 key.
struct Place {
  int c[3];
  float fr[3];
  float up[3];  // fr as seen from the upper faces of cells: the last cell has none below the points

  SGR_HD void set(const GridInfo& G, const float4& q) {
    const float qv[3] = {q.x, q.y, q.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      fr[a] = (float)(((double)qv[a] - (double)G.lo[a]) * G.inv_h - (double)c[a]);
      up[a] = fminf(fr[a], 1.f);
    }
  }
  // After set(), for a query that may lie above the points' box (and the cells):
  // as far above its cell as above these.
  SGR_HD void set_above(const GridInfo& G, const float4& q) {
    const float qv[3] = {q.x, q.y, q.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double above = ((double)qv[a] - (double)G.lo[a]) * G.inv_h - fmax((double)G.dims[a], G.ext[a] * G.inv_h);
      if (above > 0.0) up[a] = 1.f + (float)above;
    }
  }
  // distance to the slabs of cells [d, d + n) beyond the query's along axis a
  SGR_HD float gap(int a, int d, int n = 1) const {
    return fmaxf(0.f, fmaxf((float)d - fr[a], up[a] - (float)(d + n)) - 1e-3f);
  }
};

// What is left of a squared distance once that to a row is taken off, as a
// distance along the row with its margin.  Not a number where both overflowed
// (a query 1e19 cells away): the whole row then.
SGR_HD float row_reach(float left) { return left < 1e30f ? sqrtf(left) * 1.0001f + 2e-3f : INFINITY; }

// Whole cells in a distance along a row, which has at most 2^24.
SGR_HD int cell_step(float d) { return (int)floorf(fminf(3e7f, fmaxf(-3e7f, d))); }

// First of the grid's slabs of cells within R of the query's along an axis,
// counted from the query's, and their number (of a large cube, which may lie
// outside the grid nearly everywhere).
SGR_HDI int slabs(int c, int dim, int R, int& n) {
  const int first = max2(-R, -c);
  n = min2(R, dim - 1 - c) - first + 1;
  return first;
}

// Cells [xl, xr] of the row of cells (dy, dz) from the query's, within R cells
// of it and within sqrt(reach2) of the query (cell units); false: none.
SGR_HDI bool row_cells(const GridInfo& G, const Place& at, int R, int dy, int dz, float reach2, int& xl, int& xr) {
  const int cx = at.c[0], cy = at.c[1] + dy, cz = at.c[2] + dz;
  if (!(cz >= 0 && cz < G.dims[2] && cy >= 0 && cy < G.dims[1])) return false;
  const float gy = at.gap(1, dy), gz = at.gap(2, dz);
  const float left = reach2 - (gy * gy + gz * gz);
  if (left < 0.f) return false;
  // cells of the row within sqrt(left) of the query
  const float reach = row_reach(left);
  xl = max2(max2(0, cx - R), min2(cx, cx + cell_step(at.fr[0] - reach)));
  xr = min2(min2(G.dims[0] - 1, cx + R), max2(cx, cx + cell_step(at.fr[0] + reach)));
  return true;
}

// Keys below this bound belong to points nearer than every cell outside the
// cube of radius r around the query's; KEY_INF when no cell lies outside it.
SGR_HD uint64_t cube_bound(const GridInfo& G, const Place& at, int r) {
  float lb = INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (at.c[a] - r > 0) lb = fminf(lb, at.fr[a] + (float)r);
    if (at.c[a] + r < G.dims[a] - 1) lb = fminf(lb, 1.f - at.fr[a] + (float)r);
  }
  if (lb == INFINITY) return KEY_INF;
  const float d = fmaxf(0.f, lb - 1e-3f) * G.h;
  return (uint64_t)__builtin_bit_cast(uint32_t, d * d * (1.f - 2e-5f)) << 32;
}

// Radius of the smallest cube of cells around the query's outside of which no
// key below the bound lies.
SGR_HD int cells_reached(const GridInfo& G, const Place& at, uint64_t bound, int rmax) {
  const float u = sqrtf(key_of(bound)) * (float)G.inv_h * 1.0001f + 2e-3f;
  if (!(u < 1e9f)) return rmax;
  float r = 0.f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (at.c[a] > 0) r = fmaxf(r, -floorf(at.fr[a] - u));
    if (at.c[a] < G.dims[a] - 1) r = fmaxf(r, floorf(at.fr[a] + u));
  }
  return r < (float)rmax ? (int)r : rmax;
}

// A search around a query that is widened until it has found enough: all keys
// below reach2, which starts above 0 (the square of a cell may have underflowed)
// and grows 2.5 times a turn, so that it ends at the latest when it reaches the
// whole grid (last).  Returns the radius of its cube of cells.
SGR_HD float widen_first(uint64_t edge) { return fmaxf(2.f * key_of(edge), 1.1754944e-38f); }
constexpr float WIDEN = 2.5f;
SGR_HD int widen(const GridInfo& G, const Place& at, float reach2, int rmax, uint64_t& bound, bool& last) {
  bound = (uint64_t)__builtin_bit_cast(uint32_t, reach2) << 32;
  const int R = cells_reached(G, at, bound, rmax);
  last = R >= rmax;
  if (last) bound = KEY_INF;
  return R;
}

// Blocks of BLK^3 cells, listed where they hold points: what a query far from
// everything looks at instead of the cells between.
constexpr int BLK = 8;

SGR_HD int block_count(const GridInfo& G) {
  return ((G.dims[0] + BLK - 1) / BLK) * ((G.dims[1] + BLK - 1) / BLK) * ((G.dims[2] + BLK - 1) / BLK);
}

// Squared distance (cell units, never too large) from the query to the block of
// cells bc.
SGR_HDI float block_gap(const Place& at, const int bc[3]) {
  float g2 = 0.f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float g = at.gap(a, bc[a] * BLK - at.c[a], BLK);
    g2 += g * g;
  }
  return g2;
}

// Cells [xl, xr] of row r (of BLK^2) of the block bc within sqrt(reach2) of the
// query, in the grid's row (cy, cz); false: none.
SGR_HDI bool block_row_cells(const GridInfo& G, const Place& at, const int bc[3], int r, float reach2, int& cy, int& cz,
                             int& xl, int& xr) {
  cy = bc[1] * BLK + r % BLK;
  cz = bc[2] * BLK + r / BLK;
  const int x0 = bc[0] * BLK;
  if (!(cy < G.dims[1] && cz < G.dims[2])) return false;
  const float gy = at.gap(1, cy - at.c[1]), gz = at.gap(2, cz - at.c[2]);
  const float left = reach2 - (gy * gy + gz * gz);
  if (left < 0.f) return false;
  const float reach = row_reach(left);
  xl = max2(x0, at.c[0] + cell_step(at.up[0] - reach));
  xr = min2(min2(G.dims[0], x0 + BLK) - 1, at.c[0] + cell_step(at.fr[0] + reach));
  return xl <= xr;
}

}  // namespace sgr

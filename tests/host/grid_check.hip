// Host harness for the neighbour search's bounds: a serial search of the grid
// with the kernels' cells and bounds (csrc/grid_geom.h), in their order of
// places, whose bound is lowered after every row of cells, the most that any
// order of the lanes can do.
//   grid_check knn n k step     stdin: n points; lists of every step-th point
//   grid_check nn n nq tau      stdin: n points, nq queries; nearest points
// Points are float32 triples, results int32, both binary.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <vector>

#include "../../paper_1902_01061_amd/csrc/grid_geom.h"

using namespace sgr;

struct Grid {
  GridInfo G;
  std::vector<int> starts, blocks;
  std::vector<float4> pts;  // in cell order, w = index
  std::vector<int> cell;    // packed

  Grid(const std::vector<float>& p, int n, float occ, float reach) {
    float box[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int i = 0; i < n; ++i)
      for (int a = 0; a < 3; ++a) {
        box[a] = std::min(box[a], p[3 * i + a]);
        box[3 + a] = std::max(box[3 + a], p[3 * i + a]);
      }
    int cells = std::min(73728, std::max(1024, 4 * n));  // one block's
    if (n > 8192)
      for (cells = 1024; cells < 4 * n;) cells *= 2;
    G = grid_trial(box, n, cells);
    std::vector<int> cnt(G.ncells, 0);
    for (int i = 0; i < n; ++i) ++cnt[cell_index(G, p[3 * i], p[3 * i + 1], p[3 * i + 2])];
    double mu = 0;
    for (int c : cnt) mu += (double)c * c / n;
    grid_resize(G, mu, occ, reach, cells);
    starts.assign(G.ncells + 1, 0);
    for (int i = 0; i < n; ++i) ++starts[1 + cell_index(G, p[3 * i], p[3 * i + 1], p[3 * i + 2])];
    for (int c = 0; c < G.ncells; ++c) starts[c + 1] += starts[c];
    std::vector<int> at(starts.begin(), starts.end() - 1);
    pts.resize(n);
    cell.resize(n);
    for (int i = 0; i < n; ++i) {
      int c[3];
      cell_of_point(G, p[3 * i], p[3 * i + 1], p[3 * i + 2], c);
      const int j = at[cell_index(G, c)]++;
      pts[j] = make_float4(p[3 * i], p[3 * i + 1], p[3 * i + 2], __builtin_bit_cast(float, i));
      cell[j] = pack_cell(G, c);
    }
    const int b0 = (G.dims[0] + BLK - 1) / BLK, b1 = (G.dims[1] + BLK - 1) / BLK;
    for (int b = 0; b < block_count(G); ++b) {
      const int bc[3] = {b % b0, b / b0 % b1, b / (b0 * b1)};
      bool any = false;
      for (int z = bc[2] * BLK; z < std::min(G.dims[2], bc[2] * BLK + BLK); ++z)
        for (int y = bc[1] * BLK; y < std::min(G.dims[1], bc[1] * BLK + BLK); ++y) {
          const int row = (z * G.dims[1] + y) * G.dims[0];
          any |= starts[row + std::min(G.dims[0], bc[0] * BLK + BLK)] > starts[row + bc[0] * BLK];
        }
      if (any) blocks.push_back(pack_cell(G, bc));
    }
  }
};

static uint64_t key(const float4& P, const float4& q) {
  const float x = P.x - q.x, y = P.y - q.y, z = P.z - q.z;
  return (uint64_t)__builtin_bit_cast(uint32_t, (x * x + y * y) + z * z) << 32 | __builtin_bit_cast(uint32_t, P.w);
}

struct Search {
  const Grid& g;
  float4 q;
  Place at;
  int k;
  uint64_t bound;
  std::vector<uint64_t> list;
  int seen = 0;

  void span(int a, int b) {
    seen += std::max(0, b - a);
    for (int j = a; j < b; ++j) {
      const uint64_t w = key(g.pts[j], q);
      if (w < bound) list.push_back(w);
    }
    lower();
  }
  void lower() {
    if ((int)list.size() < k) return;
    std::sort(list.begin(), list.end());
    list.resize(k);
    bound = std::min(bound, list[k - 1] + 1);
  }
  void visit(int R, int inner) {
    const float inv_h = (float)g.G.inv_h;
    int ny, nz;
    const int y0 = slabs(at.c[1], g.G.dims[1], R, ny), z0 = slabs(at.c[2], g.G.dims[2], R, nz);
    for (int dz = z0; dz < z0 + nz; ++dz)
      for (int dy = y0; dy < y0 + ny; ++dy) {
        int xl, xr;
        if (!row_cells(g.G, at, R, dy, dz, key_of(bound) * (inv_h * inv_h) * (1.f + 2e-5f), xl, xr)) continue;
        const int cx = at.c[0];
        const int* st = g.starts.data() + ((at.c[2] + dz) * g.G.dims[1] + at.c[1] + dy) * g.G.dims[0];
        if (std::max(std::abs(dy), std::abs(dz)) > inner) {
          span(st[xl], st[xr + 1]);
        } else {
          if (xl < cx - inner) span(st[xl], st[cx - inner]);
          if (xr > cx + inner) span(st[cx + inner + 1], st[xr + 1]);
        }
      }
  }
  void visit_blocks() {
    const float inv_h2 = (float)g.G.inv_h * (float)g.G.inv_h * (1.f + 2e-5f);
    std::vector<std::pair<float, int>> order;
    for (int pb : g.blocks) {
      int bc[3];
      unpack_cell(g.G, pb, bc);
      order.push_back({block_gap(at, bc), pb});
    }
    std::sort(order.begin(), order.end());
    for (auto& [g2, pb] : order) {
      if (g2 > key_of(bound) * inv_h2) continue;
      int bc[3];
      unpack_cell(g.G, pb, bc);
      for (int r = 0; r < BLK * BLK; ++r) {
        int cy, cz, xl, xr;
        if (!block_row_cells(g.G, at, bc, r, key_of(bound) * inv_h2, cy, cz, xl, xr)) continue;
        const int* st = g.starts.data() + (cz * g.G.dims[1] + cy) * g.G.dims[0];
        span(st[xl], st[xr + 1]);
      }
    }
  }
};

static int rmax_of(const GridInfo& G) { return std::max(G.dims[0], std::max(G.dims[1], G.dims[2])); }

// knn_kernel and knn_far_kernel for the point at place t of the sorted array.
static std::vector<uint64_t> knn(const Grid& g, int t, int k) {
  Search s{g, g.pts[t], {}, k, 0, {}};
  unpack_cell(g.G, g.cell[t], s.at.c);
  s.at.set(g.G, s.q);
  const int own = cell_index(g.G, s.at.c);
  const bool dense = g.starts[own + 1] - g.starts[own] >= k;
  const uint64_t edge = cube_bound(g.G, s.at, 1);
  s.bound = dense ? KEY_INF : edge;
  s.visit(dense ? 0 : 1, -1);
  if (dense) {
    s.bound = std::min(s.bound, edge);
    s.visit(1, 0);
  }
  const int under = (int)std::count_if(s.list.begin(), s.list.end(), [&](uint64_t w) { return w < edge; });
  if (edge == KEY_INF || (dense ? under : (int)s.list.size()) >= k) return s.list;
  const int rmax = rmax_of(g.G);
  if (s.seen >= k) {
    float reach2 = widen_first(edge);
    for (int round = 0; round < 1000; ++round, reach2 *= WIDEN) {
      bool last;
      s.list.clear();
      const int R = widen(g.G, s.at, reach2, rmax, s.bound, last);
      s.visit(R, -1);
      if ((int)s.list.size() >= k || last) return s.list;
    }
    std::fprintf(stderr, "no end\n");
    std::exit(1);
  }
  s.list.clear();
  s.bound = KEY_INF;
  const int n = (int)g.pts.size(), first = std::max(0, std::min(t - 64, n - 128));
  s.span(first, std::min(n, first + 128));
  s.list.clear();
  for (int inner = -1, R = 3; R <= 18; R = 2 * R + 2) {
    R = std::min(R, cells_reached(g.G, s.at, s.bound, rmax));
    if (R <= inner) return s.list;
    s.visit(R, inner);
    inner = R;
  }
  if (cells_reached(g.G, s.at, s.bound, rmax) <= 18) return s.list;
  s.list.clear();
  s.visit_blocks();
  return s.list;
}

// nearest_kernel and nearest_far_kernel.
static int nearest(const Grid& g, const float4& q, float max_key) {
  const uint64_t top = (uint64_t)__builtin_bit_cast(uint32_t, max_key) << 32 | 0xffffffffu;
  Search s{g, q, {}, 1, top, {}};
  cell_of_point(g.G, q.x, q.y, q.z, s.at.c);
  s.at.set(g.G, q);
  bool found;
  for (int inner = -1, R = 0;;) {
    s.visit(R, inner);
    const int want = cells_reached(g.G, s.at, s.bound, 1 << 20);
    found = want <= R || cube_bound(g.G, s.at, R) == KEY_INF;
    if (found || (R > 0 && want > 3)) break;
    inner = R;
    R = R == 0 ? 1 : want;
  }
  if (!found) {
    s.at.set_above(g.G, q);
    const int n = (int)g.pts.size(), first = std::max(0, std::min(g.starts[cell_index(g.G, s.at.c)] - 32, n - 64));
    s.list.clear();
    s.bound = top;
    s.span(first, std::min(n, first + 64));
    if (cells_reached(g.G, s.at, s.bound, 1 << 20) <= 6)
      s.visit(6, -1);
    else
      s.visit_blocks();
  }
  return !s.list.empty() && key_of(s.list[0]) < INFINITY && key_of(s.list[0]) <= max_key ? (int)(uint32_t)s.list[0] : -1;
}

static std::vector<float> points(int n) {
  std::vector<float> p(3 * (size_t)n);
  if (std::fread(p.data(), 12, n, stdin) != (size_t)n) std::exit(2);
  return p;
}

int main(int argc, char** argv) {
  const bool lists = !std::strcmp(argv[1], "knn");
  const int n = std::atoi(argv[2]), m = std::atoi(argv[3]);
  const std::vector<float> p = points(n);
  if (lists) {
    const int step = std::atoi(argv[4]);
    const Grid g(p, n, std::max(2.0f, 0.5f * (float)m), 0.f);
    std::vector<int> out(((n - 1) / step + 1) * (size_t)m, -1);
    for (int t = 0; t < n; ++t) {
      const int i = __builtin_bit_cast(int, g.pts[t].w);
      if (i % step) continue;
      std::vector<uint64_t> l = knn(g, t, m);
      std::sort(l.begin(), l.end());
      for (int e = 0; e < std::min(m, (int)l.size()); ++e) out[(size_t)(i / step) * m + e] = (int)(uint32_t)l[e];
    }
    std::fwrite(out.data(), 4, out.size(), stdout);
  } else {
    const std::vector<float> qs = points(m);
    const float tau = (float)std::atof(argv[4]), max_key = tau * tau;
    const Grid g(p, n, 4.f, std::min(1e30f, 1.002f * std::sqrt(max_key)));
    std::vector<int> out(m);
    for (int i = 0; i < m; ++i) out[i] = nearest(g, make_float4(qs[3 * i], qs[3 * i + 1], qs[3 * i + 2], 0.f), max_key);
    std::fwrite(out.data(), 4, m, stdout);
  }
}

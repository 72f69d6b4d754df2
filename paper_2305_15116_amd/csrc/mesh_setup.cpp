// Host set-up of a macro mesh: topology, per-level stencils and element
// matrices, interface groups, tile lists, coarse direct solver, device upload.
//
// The macro mesh is the unstructured coarse grid of the paper; each macro is
// refined uniformly, giving a structured index space per macro (Intro,
// "Hybrid Tetrahedral Grids").  Because all interior rows of a macro are the
// same, one stencil per macro and level is computed here (the paper's
// constant stencils, PETSc comparison section) from the element matrices of
// the few micro-element types; DoFs on macro boundaries are gathered into
// "groups" (one per unique DoF) that the interface kernel completes.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <string>
#include <thread>
#include <vector>

#include "mesh.hpp"

namespace mf {

namespace {
thread_local std::string t_err;
}

int set_error(int code, const std::string& msg) {
  t_err = msg;
  return code;
}
const char* last_error() { return t_err.c_str(); }

namespace {

// Element matrix of a simplex with edge matrix E (columns = edges from vertex
// 0) via the metric tensor: with G = E^{-T} the barycentric gradients of
// vertices 1..d are the columns of G, so g_i . g_j = ((E^T E)^{-1})_ij;
// vertex 0's gradient is minus their sum.  K = |T| (g_i . g_j).
bool metric_stiffness(int dim, const double E[3][3], double K[4][4]) {
  double Mt[3][3] = {{0}};
  for (int i = 0; i < dim; ++i)
    for (int j = 0; j < dim; ++j) {
      double s = 0.0;
      for (int r = 0; r < dim; ++r) s += E[r][i] * E[r][j];
      Mt[i][j] = s;
    }
  double det, inv[3][3] = {{0}};
  if (dim == 2) {
    det = Mt[0][0] * Mt[1][1] - Mt[0][1] * Mt[1][0];
    if (!(det > 0.0)) return false;
    inv[0][0] = Mt[1][1] / det;
    inv[1][1] = Mt[0][0] / det;
    inv[0][1] = inv[1][0] = -Mt[0][1] / det;
  } else {
    const double a = Mt[0][0], b = Mt[0][1], c = Mt[0][2], d = Mt[1][1], e = Mt[1][2], f = Mt[2][2];
    const double A = d * f - e * e, B = c * e - b * f, C = b * e - c * d;
    det = a * A + b * B + c * C;
    if (!(det > 0.0)) return false;
    inv[0][0] = A / det;
    inv[0][1] = inv[1][0] = B / det;
    inv[0][2] = inv[2][0] = C / det;
    inv[1][1] = (a * f - c * c) / det;
    inv[1][2] = inv[2][1] = (b * c - a * e) / det;
    inv[2][2] = (a * d - b * b) / det;
  }
  // |det E| = sqrt(det(E^T E))
  const double vol = std::sqrt(det) / (dim == 2 ? 2.0 : 6.0);
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) K[i][j] = 0.0;
  for (int i = 0; i < dim; ++i)
    for (int j = 0; j < dim; ++j) K[i + 1][j + 1] = vol * inv[i][j];
  for (int j = 1; j <= dim; ++j) {
    double s = 0.0;
    for (int i = 1; i <= dim; ++i) s += K[i][j];
    K[0][j] = -s;
    K[j][0] = -s;
  }
  double s = 0.0;
  for (int i = 1; i <= dim; ++i)
    for (int j = 1; j <= dim; ++j) s += K[i][j];
  K[0][0] = s;
  return true;
}

struct PointKey {
  int64_t v[4];
  int32_t w[4];
  bool operator<(const PointKey& o) const {
    for (int k = 0; k < 4; ++k) {
      if (v[k] != o.v[k]) return v[k] < o.v[k];
      if (w[k] != o.w[k]) return w[k] < o.w[k];
    }
    return false;
  }
  bool operator==(const PointKey& o) const {
    for (int k = 0; k < 4; ++k)
      if (v[k] != o.v[k] || w[k] != o.w[k]) return false;
    return true;
  }
};

PointKey point_key(int dim, const int64_t* cellv, int N, int x, int y, int z) {
  const int64_t w[4] = {N - x - y - (dim == 3 ? z : 0), x, y, z};
  std::pair<int64_t, int64_t> pr[4];
  int n = 0;
  for (int k = 0; k <= dim; ++k)
    if (w[k] != 0) pr[n++] = {cellv[k], w[k]};
  // insertion sort by vertex id (at most 4 entries)
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && pr[j].first < pr[j - 1].first; --j) std::swap(pr[j], pr[j - 1]);
  PointKey k;
  for (int i = 0; i < 4; ++i) {
    k.v[i] = i < n ? pr[i].first : -1;
    k.w[i] = i < n ? (int32_t)pr[i].second : 0;
  }
  return k;
}

template <class F>
void for_each_boundary_point(int dim, int N, F&& fn) {
  if (dim == 2) {
    for (int y = 0; y <= N; ++y) {
      if (y == 0 || y == N) {
        for (int x = 0; x <= N - y; ++x) fn(x, y, 0);
      } else {
        fn(0, y, 0);
        fn(N - y, y, 0);
      }
    }
    return;
  }
  for (int z = 0; z <= N; ++z) {
    const int M = N - z;
    for (int y = 0; y <= M; ++y) {
      if (z == 0 || y == 0 || y == M) {
        for (int x = 0; x <= M - y; ++x) fn(x, y, z);
      } else {
        fn(0, y, z);
        fn(M - y, y, z);
      }
    }
  }
}

// Runs fn(i) for i in [0, n) on up to 16 host threads when `work` is large.
template <class F>
void parallel_for(size_t n, int64_t work, F&& fn) {
  unsigned nt = std::min(16u, std::max(1u, std::thread::hardware_concurrency()));
  if (work < (1 << 20) || n < 2) nt = 1;
  nt = (unsigned)std::min<size_t>(nt, n);
  if (nt <= 1) {
    for (size_t i = 0; i < n; ++i) fn(i);
    return;
  }
  std::atomic<size_t> next{0};
  std::vector<std::thread> th;
  for (unsigned t = 0; t < nt; ++t)
    th.emplace_back([&] {
      for (size_t i; (i = next.fetch_add(1)) < n;) fn(i);
    });
  for (auto& t : th) t.join();
}

// Points whose support is exactly a primitive of p vertices.
int64_t prim_points(int N, int p) {
  if (p == 1) return 1;
  if (p == 2) return std::max(N - 1, 0);
  return N >= 2 ? (int64_t)(N - 1) * (N - 2) / 2 : 0;
}

}  // namespace

// ---------------------------------------------------------------- topology
static int build_topology(mf_mesh* m) {
  const int d1 = m->dim + 1;
  std::map<std::vector<int64_t>, int> facet_count;
  std::map<std::vector<int64_t>, int64_t> seen;
  for (int64_t c = 0; c < m->nc; ++c) {
    std::vector<int64_t> s(&m->cells[c * d1], &m->cells[c * d1] + d1);
    std::sort(s.begin(), s.end());
    for (int k = 0; k + 1 < d1; ++k)
      if (s[k] == s[k + 1]) return set_error(MF_EINVAL, "cell " + std::to_string(c) + " repeats a vertex");
    if (seen.count(s)) return set_error(MF_EINVAL, "cell " + std::to_string(c) + " repeats an earlier cell");
    seen[s] = c;
    for (int skip = 0; skip < d1; ++skip) {
      std::vector<int64_t> f;
      for (int k = 0; k < d1; ++k)
        if (k != skip) f.push_back(s[k]);
      if (++facet_count[f] > 2) return set_error(MF_EINVAL, "non-conforming mesh: a facet has more than two cells");
    }
  }
  // lowest macro containing each primitive (vertex subset of a cell), and how many contain it
  std::map<std::vector<int64_t>, int64_t> owner;
  std::map<std::vector<int64_t>, int> containing;
  for (int64_t c = 0; c < m->nc; ++c)
    for (int s = 1; s < (1 << d1); ++s) {
      std::vector<int64_t> prim;
      for (int k = 0; k < d1; ++k)
        if (s & (1 << k)) prim.push_back(m->cells[c * d1 + k]);
      std::sort(prim.begin(), prim.end());
      auto it = owner.find(prim);
      if (it == owner.end() || it->second > c) owner[prim] = c;
      containing[prim] += 1;
    }
  // primitives lying in a boundary facet
  std::map<std::vector<int64_t>, bool> on_boundary;
  for (auto& kv : facet_count) {
    if (kv.second != 1) continue;
    const auto& f = kv.first;
    const int n = (int)f.size();
    for (int s = 1; s < (1 << n); ++s) {
      std::vector<int64_t> prim;
      for (int k = 0; k < n; ++k)
        if (s & (1 << k)) prim.push_back(f[k]);
      on_boundary[prim] = true;
    }
  }
  const bool dirichlet = (m->flags & MF_FLAG_DIRICHLET) != 0;
  m->own_mask.assign(m->nc, 0);
  m->dir_mask.assign(m->nc, 0);
  m->shared_mask.assign(m->nc, 0);
  for (int64_t c = 0; c < m->nc; ++c)
    for (int s = 1; s < (1 << d1); ++s) {
      std::vector<int64_t> prim;
      for (int k = 0; k < d1; ++k)
        if (s & (1 << k)) prim.push_back(m->cells[c * d1 + k]);
      std::sort(prim.begin(), prim.end());
      if (owner[prim] == c) m->own_mask[c] |= (uint16_t)(1u << s);
      if (containing[prim] >= 2) m->shared_mask[c] |= (uint16_t)(1u << s);
      if (dirichlet && on_boundary.count(prim)) m->dir_mask[c] |= (uint16_t)(1u << s);
    }
  // every proper vertex subset of a cell is a macro-boundary primitive
  m->prims.clear();
  std::map<std::vector<int64_t>, size_t> index;
  for (auto& kv : containing) {
    if ((int)kv.first.size() == d1) continue;
    index[kv.first] = m->prims.size();
    Prim P;
    P.v = kv.first;
    P.dirichlet = dirichlet && on_boundary.count(kv.first) > 0;
    m->prims.push_back(std::move(P));
  }
  for (int64_t c = 0; c < m->nc; ++c)
    for (int s = 1; s < (1 << d1) - 1; ++s) {
      std::vector<int64_t> prim;
      for (int k = 0; k < d1; ++k)
        if (s & (1 << k)) prim.push_back(m->cells[c * d1 + k]);
      std::sort(prim.begin(), prim.end());
      Prim& P = m->prims[index.at(prim)];
      std::array<int8_t, 3> loc{};
      for (size_t j = 0; j < P.v.size(); ++j)
        for (int k = 0; k < d1; ++k)
          if (m->cells[c * d1 + k] == P.v[j]) loc[j] = (int8_t)k;
      P.cell.push_back(c);  // cells are visited in increasing order
      P.local.push_back(loc);
    }
  return MF_OK;
}

// ---------------------------------------------------------------- 3D tiles
// Column tiles of every macro's slabs, padded to whole workgroups.
static std::vector<Tile> column_tiles(int N, int64_t nc, const Shape3& sh) {
  std::vector<Tile> out;
  for (int64_t c = 0; c < nc; ++c)
    for (int z0 = 1; z0 <= N - 2; z0 += sh.PZ) {
      // columns of the slab: band b has N - z0 - R b of them, as long as its first row has two
      int Q = 0;
      for (int b = 0; N - z0 - sh.R * b >= 2; ++b) Q += N - z0 - sh.R * b;
      const int nz = std::min(sh.PZ, N - 1 - z0);
      for (int q0 = -1; q0 + 1 < Q; q0 += kTileW) out.push_back({(int32_t)c, q0, Q, z0 | nz << 16});
    }
  while (out.size() % kWavesPerWG) out.push_back({-1, 0, 0, 0});
  return out;
}

// MacroDev::zinv: the assembled diagonals by macro and support.
static void set_assembled_diagonals(const mf_mesh* m, Level& L) {
  const StencilTable ST = stencil_table(m->dim);
  for (int64_t c = 0; c < m->nc; ++c) L.md[c].zinv[full_mask(m->dim)] = L.md[c].inv_diag;
  parallel_for(m->prims.size(), 512 * (int64_t)m->prims.size(), [&](size_t i) {
    const Prim& P = m->prims[i];
    auto mask = [&](size_t k) {
      int s = 0;
      for (size_t j = 0; j < P.v.size(); ++j) s |= 1 << P.local[k][j];
      return s;
    };
    double diag = 0.0;
    for (size_t k = 0; k < P.cell.size(); ++k) diag += L.md[P.cell[k]].wm[mask(k)][ST.centre];
    for (size_t k = 0; k < P.cell.size(); ++k)
      L.md[P.cell[k]].zinv[mask(k)] = P.dirichlet || diag == 0.0 ? 0.0 : 1.0 / diag;
  });
  for (int64_t c = 0; c < m->nc; ++c)
    for (int s = 0; s < 16; ++s) L.md[c].zinvf[s] = (float)L.md[c].zinv[s];
}

// Cuts DoFs of n copies each, one after the other in Level::edges, into edge tiles
// of up to 64 copies per step and `steps` steps (more than 64 copies: a tile of
// its own, kEdgeBigTile), and notes the lane of each DoF's first copy.
struct EdgeCutter {
  int steps;
  std::vector<Tile>& out;
  std::vector<uint8_t> head;
  int32_t first = 0, at = 0, n[2] = {0, 0}, step = 0;  // of the open tile; at: the next copy
  void close() {
    if (n[0] > 0) out.push_back({kEdgeTile, first, n[0], n[1]});
    first = at;
    n[0] = n[1] = step = 0;
  }
  void add(int nc) {
    if (nc > kWave) {
      close();
      at += nc;
      out.push_back({kEdgeBigTile, first, nc, 0});
      first = at;
      head.push_back(0);
      return;
    }
    if (n[step] + nc > kWave && ++step == steps) close();
    head.push_back((uint8_t)n[step]);
    at += nc;
    n[step] += nc;
  }
};

// The records of a DoF's nc copies from e on.
static void set_copies(EdgeCopy* e, int dim, int N, const Copy* k, const int64_t* idx, int nc, int head, bool dirichlet) {
  for (int c = 0; c < nc; ++c) {
    e[c].idx = idx[c];
    e[c].macro = k[c].macro;
    e[c].x = (uint16_t)k[c].x, e[c].y = (uint16_t)k[c].y, e[c].z = (uint16_t)k[c].z;
    e[c].mask = (uint8_t)support_mask(dim, N, k[c].x, k[c].y, k[c].z);
    e[c].head = (uint8_t)head;
    e[c].copies = (uint8_t)(nc > kWave ? 0 : nc);
    e[c].dirichlet = dirichlet ? 1 : 0;
  }
}

// Tiles of a 2D level's DoFs that macros share (the exchange list), at the head
// of both tile lists so that they start first.
static void build_edge_tiles2(Level& L) {
  std::vector<Tile>& out = L.tiles;
  const int64_t ng = L.nxgroups();
  EdgeCutter cut{2, out};
  cut.head.reserve(ng);
  for (int64_t g = 0; g < ng; ++g) cut.add(L.xgrp_ptr[g + 1] - L.xgrp_ptr[g]);
  cut.close();
  L.edges.resize(L.xcopies.size());
  constexpr int64_t kChunk = 1 << 12;
  parallel_for((size_t)((ng + kChunk - 1) / kChunk), 8 * (int64_t)L.edges.size(), [&](size_t k) {
    for (int64_t g = (int64_t)k * kChunk; g < std::min(ng, (int64_t)(k + 1) * kChunk); ++g) {
      const int c = L.xgrp_ptr[g];
      set_copies(&L.edges[c], 2, L.N, &L.xcopies[c], &L.xcpidx[c], L.xgrp_ptr[g + 1] - c, cut.head[g], false);
    }
  });
  L.btiles = out;
  while (out.size() % kWavesPerWG) out.push_back({-1, 0, 0, 0});
  L.ewgs = (int)(out.size() / kWavesPerWG);
  L.tiles_f32 = out;
}

// The tiles of a 2D level that is small enough for short ones (edge tiles of
// one step each).
static void build_short_tiles2(Level& L, int64_t nc) {
  constexpr size_t most = (size_t)kShortWGs * kWavesPerWG;
  std::vector<Tile>& out = L.tiles_short;
  L.short_rows = 0;
  for (int rows : kTileShort) {
    out.clear();
    for (int i = 0; i < L.ewgs * kWavesPerWG && out.size() <= most; ++i) {
      const Tile& t = L.tiles[i];
      if (t.macro == -1) continue;
      out.push_back({t.macro, t.x0, t.y0, 0});
      if (t.z > 0) out.push_back({t.macro, t.x0 + t.y0, t.z, 0});
    }
    while (out.size() % kWavesPerWG) out.push_back({-1, 0, 0, 0});
    L.ewgs_short = (int)(out.size() / kWavesPerWG);
    for (int64_t c = 0; c < nc && out.size() <= most; ++c)
      for (int y0 = 0; y0 <= L.N && out.size() <= most; y0 += rows)
        for (int x0 = 0; x0 + y0 <= L.N; x0 += kTileW) out.push_back({(int32_t)c, x0, y0, 0});
    while (out.size() % kWavesPerWG) out.push_back({-1, 0, 0, 0});
    if (out.size() <= most) {
      L.short_rows = rows;
      return;
    }
  }
  out.clear();
}

// Tiles of a 3D level: the interior walk's slabs of every macro, the inner
// points of every macro face, and the copies of the edge and vertex DoFs.
static void build_tiles3(const mf_mesh* m, Level& L) {
  const int N = L.N;
  std::vector<Tile> bnd;
  const StencilTable ST = stencil_table(3);
  L.tiles = column_tiles(N, m->nc, shape3(N));
  for (int f32 = 0; f32 < 2; ++f32) L.vtiles[f32] = column_tiles(N, m->nc, shape3_varcoef(N, f32));
  // faces: weights a and b run over two of the face's vertices, with a along
  // the first macro's x where its face holds vertices 0 and 1 (contiguous storage)
  for (const Prim& P : m->prims) {
    if (P.v.size() != 3 || N < kMinFaceN) continue;
    int pa = 0, pb = 1, pc = 2;
    for (int j = 0; j < 3; ++j) {
      if (P.local[0][j] == 1) pa = j;
      if (P.local[0][j] == 0) pc = j;
    }
    const bool lined = P.local[0][pa] == 1 && P.local[0][pc] == 0;
    if (!lined) {  // the far face or x = 0: a along y
      for (int j = 0; j < 3; ++j) {
        if (P.local[0][j] == 2) pa = j;
        if (P.local[0][j] == 3) pb = j;
      }
      pc = 3 - pa - pb;
    }
    pb = 3 - pa - pc;
    FaceDev F{};
    F.N = N;
    F.copies = (int16_t)P.cell.size();
    F.dirichlet = P.dirichlet ? 1 : 0;
    double diag = 0.0;
    for (int i = 0; i < 2; ++i) {
      const size_t k = std::min<size_t>(i, P.cell.size() - 1);
      FaceCopy& C = F.cp[i];
      C.macro = (int32_t)P.cell[k];
      int mask = 0;
      for (int j = 0; j < 3; ++j) {
        const int l = P.local[k][j];
        mask |= 1 << l;
        if (l == 0) continue;
        if (j == pa) C.a[l - 1] = 1;
        else if (j == pb) C.b[l - 1] = 1;
        else C.n[l - 1] = 1, C.a[l - 1] = C.b[l - 1] = -1;
      }
      for (int f = 0; f < 4; ++f)
        if (!((mask >> f) & 1)) C.face = (int8_t)f;
      if (k == (size_t)i) diag += L.md[C.macro].wm[mask][ST.centre];
    }
    if (F.dirichlet && F.cp[0].face <= 1) continue;  // written by the walk
    F.inv = diag != 0.0 ? 1.0 / diag : 0.0;
    F.invf = (float)F.inv;
    const int id = (int)L.faces.size(), n = (N - 1) * (N - 2) / 2;
    L.faces.push_back(F);
    auto cut = [&](std::vector<Tile>& to, const FaceRuns& r) {
      const int run = F.dirichlet ? r.dirichlet : (F.copies == 1 ? r.one : r.two);
      for (int i = 0; i < n; i += run) to.push_back({kFaceTile, i, std::min(run, n - i), id});
    };
    cut(bnd, face_runs(N));
    cut(L.btiles, kFaceRunsWG);
  }
  // edge and vertex DoFs, and on the smallest levels the inner points of the faces that the walk
  // does not write (whole primitives of the all-groups list)
  struct Range {
    size_t prim;
    int64_t n, copies, dof, edge;  // its DoFs; its first of the list's copies, of the DoFs and of the edges
  };
  std::vector<Range> ranges;
  std::vector<Tile> etiles;
  EdgeCutter cut{1, etiles};
  int64_t c0 = 0;
  for (size_t i = 0; i < m->prims.size(); ++i) {
    const Prim& P = m->prims[i];
    const int64_t n = prim_points(N, (int)P.v.size()), nc = (int64_t)P.cell.size();
    int mask = 0;
    for (size_t j = 0; j < P.v.size(); ++j) mask |= 1 << P.local[0][j];
    const bool face = P.v.size() == 3;
    if (n > 0 && !(face && N >= kMinFaceN) && !((mask == 13 || mask == 14) && P.dirichlet)) {
      ranges.push_back({i, n, c0, (int64_t)cut.head.size(), cut.at});
      for (int64_t g = 0; g < n; ++g) cut.add((int)nc);
    }
    c0 += n * nc;
  }
  cut.close();
  L.edges.resize((size_t)cut.at);
  parallel_for(ranges.size(), 8 * (int64_t)cut.at, [&](size_t r) {
    const Range& R = ranges[r];
    const Prim& P = m->prims[R.prim];
    const int64_t nc = (int64_t)P.cell.size();
    for (int64_t g = 0; g < R.n; ++g)
      set_copies(&L.edges[R.edge + g * nc], 3, N, &L.copies[R.copies + g * nc], &L.cpidx[R.copies + g * nc], (int)nc,
                 cut.head[R.dof + g], P.dirichlet);
  });
  bnd.insert(bnd.end(), etiles.begin(), etiles.end());
  L.btiles.insert(L.btiles.end(), etiles.begin(), etiles.end());
  while (bnd.size() % kWavesPerWG) bnd.push_back({-1, 0, 0, 0});
  // the boundary's workgroups are spread evenly among the walk's (each XCD
  // takes a contiguous chunk of workgroups, so appended ones would all land on one)
  const size_t nr = L.tiles.size() / kWavesPerWG, nb = bnd.size() / kWavesPerWG;
  std::vector<Tile> all;
  all.reserve(L.tiles.size() + bnd.size());
  for (size_t ir = 0, ib = 0; ir < nr || ib < nb;) {
    const bool take = ib < nb && (ir == nr || ib * nr <= ir * nb);
    const Tile* src = take ? &bnd[ib++ * kWavesPerWG] : &L.tiles[ir++ * kWavesPerWG];
    all.insert(all.end(), src, src + kWavesPerWG);
  }
  L.tiles.swap(all);
}

// ---------------------------------------------------------------- per level
static int build_level(mf_mesh* m, int level, Level& L) {
  const int dim = m->dim, d1 = dim + 1;
  const int N = 1 << level;
  L.level = level;
  L.N = N;
  const ElemTable ET = elem_table(dim);
  const StencilTable ST = stencil_table(dim);

  // storage offsets and macro constants
  L.base.resize(m->nc);
  L.md.assign(m->nc, MacroDev{});
  int64_t off = 0;
  for (int64_t c = 0; c < m->nc; ++c) {
    L.base[c] = off;
    off += macro_points(dim, N);
    MacroDev& M = L.md[c];
    std::memset(&M, 0, sizeof(M));
    M.base = L.base[c];
    for (int k = 0; k < 4; ++k) M.vid[k] = k < d1 ? m->cells[c * d1 + k] : -1;
    M.N = N;
    M.own_mask = m->own_mask[c];
    M.dir_mask = m->dir_mask[c];
    M.shared_mask = m->shared_mask[c];
    // macro Jacobian columns P_k - P_0
    const double* P0 = &m->coords[m->cells[c * d1] * dim];
    double J[3][3] = {{0}};
    for (int k = 1; k <= dim; ++k) {
      const double* Pk = &m->coords[m->cells[c * d1 + k] * dim];
      for (int r = 0; r < dim; ++r) J[r][k - 1] = Pk[r] - P0[r];
    }
    for (int t = 0; t < ET.ntypes; ++t) {
      double E[3][3] = {{0}};
      for (int k = 1; k <= dim; ++k)
        for (int r = 0; r < dim; ++r) {
          double s = 0.0;
          for (int q = 0; q < dim; ++q) s += J[r][q] * (double)(ET.off[t][k][q] - ET.off[t][0][q]);
          E[r][k - 1] = s / (double)N;
        }
      double K[4][4];
      if (!metric_stiffness(dim, E, K)) return set_error(MF_EINVAL, "degenerate macro " + std::to_string(c));
      for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) {
          M.K[t][i * 4 + j] = K[i][j];
          M.Kf[t][i * 4 + j] = (float)K[i][j];
        }
    }
    // Partial stencil of every support mask: sum, over the (type, local vertex v)
    // incidences of the micro-elements inside the macro that contain a point
    // with that support, of row v of K_t.  An incidence is present iff the
    // element's vertex offset o_v is zero in every coordinate that vanishes
    // at the point, and, on the far face (weight w0 = 0), iff o_v has the
    // largest coordinate sum of its type; the full mask gives the interior stencil.
    const int fm = full_mask(dim);
    for (int mask = 1; mask <= fm; ++mask) {
      for (int t = 0; t < ET.ntypes; ++t)
        for (int v = 0; v < ET.nv; ++v) {
          bool ok = true;
          int osum = 0;
          for (int k = 0; k < dim; ++k) {
            osum += ET.off[t][v][k];
            if (!((mask >> (k + 1)) & 1) && ET.off[t][v][k] != 0) ok = false;
          }
          if (!(mask & 1) && osum != ET.slack[t]) ok = false;
          if (!ok) continue;
          for (int u = 0; u < ET.nv; ++u) {
            int d[3] = {0, 0, 0};
            for (int k = 0; k < 3; ++k) d[k] = ET.off[t][u][k] - ET.off[t][v][k];
            int hit = -1;
            for (int q = 0; q < ST.n; ++q)
              if (ST.off[q][0] == d[0] && ST.off[q][1] == d[1] && ST.off[q][2] == d[2]) hit = q;
            if (hit < 0) return set_error(MF_EINVAL, "internal: stencil offset not found");
            M.wm[mask][hit] += M.K[t][v * 4 + u];
          }
        }
      for (int q = 0; q < ST.n; ++q) M.wmf[mask][q] = (float)M.wm[mask][q];
    }
    M.inv_diag = 1.0 / M.wm[fm][ST.centre];
    M.inv_diagf = (float)M.inv_diag;
  }
  L.storage = off;

  // interface groups: every macro-boundary DoF, primitive by primitive (the
  // points whose support is exactly that vertex / edge / face), with one copy
  // per containing macro in macro order.  Offsets are counted first, then the
  // primitives are filled in parallel.
  const size_t np = m->prims.size();
  std::vector<int64_t> g_off(np + 1, 0), c_off(np + 1, 0), x_off(np + 1, 0), xc_off(np + 1, 0);
  for (size_t i = 0; i < np; ++i) {
    const Prim& P = m->prims[i];
    const int64_t n = prim_points(N, (int)P.v.size()), nc = (int64_t)P.cell.size();
    const bool xg = !P.dirichlet && nc >= 2;
    g_off[i + 1] = g_off[i] + n;
    c_off[i + 1] = c_off[i] + n * nc;
    x_off[i + 1] = x_off[i] + (xg ? n : 0);
    xc_off[i + 1] = xc_off[i] + (xg ? n * nc : 0);
  }
  if (c_off[np] > (int64_t)INT32_MAX) return set_error(MF_ENOMEM, "too many interface copies");
  L.grp_ptr.assign(g_off[np] + 1, 0);
  L.grp_flag.assign(g_off[np], 0);
  L.copies.assign(c_off[np], Copy{});
  L.xgrp_ptr.assign(x_off[np] + 1, 0);
  L.xcopies.assign(xc_off[np], Copy{});
  L.xgrp_invdiag.assign(x_off[np], 0.0);
  L.grp_ptr[g_off[np]] = (int32_t)c_off[np];
  L.xgrp_ptr[x_off[np]] = (int32_t)xc_off[np];
  auto fill = [&](size_t i) {
    const Prim& P = m->prims[i];
    const int p = (int)P.v.size();
    const size_t nc = P.cell.size();
    const bool xg = !P.dirichlet && nc >= 2;
    int64_t g = g_off[i], c = c_off[i], xi = x_off[i], xc = xc_off[i];
    auto emit = [&](const int* w) {
      L.grp_ptr[g] = (int32_t)c;
      L.grp_flag[g] = P.dirichlet ? 1 : 0;
      ++g;
      double diag = 0.0;
      if (xg) L.xgrp_ptr[xi] = (int32_t)xc;
      for (size_t k = 0; k < nc; ++k) {
        int wl[4] = {0, 0, 0, 0};
        for (int j = 0; j < p; ++j) wl[P.local[k][j]] = w[j];
        const Copy cp{(int32_t)P.cell[k], wl[1], wl[2], dim == 3 ? wl[3] : 0};
        L.copies[c++] = cp;
        if (xg) {
          L.xcopies[xc++] = cp;
          // the assembled diagonal is the sum of the copies' partial centre weights
          diag += L.md[cp.macro].wm[support_mask(dim, N, cp.x, cp.y, cp.z)][ST.centre];
        }
      }
      if (xg) L.xgrp_invdiag[xi++] = diag != 0.0 ? 1.0 / diag : 0.0;
    };
    int w[3];
    if (p == 1) {
      w[0] = N;
      emit(w);
    } else if (p == 2) {
      for (w[0] = 1; w[0] <= N - 1; ++w[0]) {
        w[1] = N - w[0];
        emit(w);
      }
    } else {
      for (w[0] = 1; w[0] <= N - 2; ++w[0])
        for (w[1] = 1; w[0] + w[1] <= N - 1; ++w[1]) {
          w[2] = N - w[0] - w[1];
          emit(w);
        }
    }
  };
  parallel_for(np, c_off[np], fill);
  const int64_t ngroups = L.ngroups();
  // unique DoFs: interior points of every macro + groups
  int64_t interior = 0;
  if (dim == 2) interior = N >= 3 ? tri_count(N - 2) : 0;
  else interior = N >= 4 ? tet_count(N - 3) : 0;
  L.unique = interior * m->nc + ngroups;

  // owner bits: bit i set iff storage DoF i is the copy that counts its
  // unique DoF in norms and dot products (interior points, and boundary
  // points whose primitive this macro owns)
  // (slices of every macro on several threads: a word whose bits come from
  // two rows is or-ed atomically, words inside one row are stored)
  std::vector<std::atomic<uint32_t>> bits((size_t)((L.storage + 31) / 32));
  for (auto& w : bits) w.store(0u, std::memory_order_relaxed);
  auto set_range = [&](int64_t lo, int64_t hi) {  // bits [lo, hi)
    for (int64_t i = lo; i < hi;) {
      if ((i & 31) == 0 && i + 32 <= hi) {
        bits[i >> 5].store(0xffffffffu, std::memory_order_relaxed);
        i += 32;
      } else {
        bits[i >> 5].fetch_or(1u << (i & 31), std::memory_order_relaxed);
        ++i;
      }
    }
  };
  const int nz = dim == 3 ? N + 1 : 1;
  parallel_for((size_t)(m->nc * nz), L.storage, [&](size_t job) {
    const int64_t c = (int64_t)job / nz;
    const int z = (int)((int64_t)job % nz);
    const uint16_t om = m->own_mask[c];
    const int S = N - z;
    for (int y = 0; y <= S; ++y) {
      const int64_t r0 = L.base[c] + (dim == 2 ? idx2(N, 0, y) : idx3(N, 0, y, z));
      const int len = S - y + 1;
      if (y >= 1 && z >= 1 - (dim == 2 ? 1 : 0) && len >= 3) {
        set_range(r0 + 1, r0 + len - 1);
        for (int x : {0, len - 1})
          if ((om >> support_mask(dim, N, x, y, z)) & 1) set_range(r0 + x, r0 + x + 1);
      } else {
        for (int x = 0; x < len; ++x) {
          const int mk = support_mask(dim, N, x, y, z);
          if (mk == full_mask(dim) || ((om >> mk) & 1)) set_range(r0 + x, r0 + x + 1);
        }
      }
    }
  });
  L.own_bits.resize(bits.size());
  for (size_t i = 0; i < bits.size(); ++i) L.own_bits[i] = bits[i].load(std::memory_order_relaxed);

  // storage indices of the copies, so that kernels index directly
  auto storage_index = [&](const Copy& c) {
    return L.md[c.macro].base + (dim == 2 ? idx2(N, c.x, c.y) : idx3(N, c.x, c.y, c.z));
  };
  L.cpidx.resize(L.copies.size());
  L.xcpidx.resize(L.xcopies.size());
  constexpr size_t kChunk = 1 << 16;
  parallel_for((L.copies.size() + kChunk - 1) / kChunk, (int64_t)L.copies.size(), [&](size_t k) {
    for (size_t i = k * kChunk; i < std::min(L.copies.size(), (k + 1) * kChunk); ++i) L.cpidx[i] = storage_index(L.copies[i]);
  });
  parallel_for((L.xcopies.size() + kChunk - 1) / kChunk, (int64_t)L.xcopies.size(), [&](size_t k) {
    for (size_t i = k * kChunk; i < std::min(L.xcopies.size(), (k + 1) * kChunk); ++i)
      L.xcpidx[i] = storage_index(L.xcopies[i]);
  });

  // wave tiles, natural order: 2D the copies of shared DoFs, then every point
  // of every macro (macro, band, strip); 3D over the interior points (macro, slab, columns), then the
  // macro faces and the edge and vertex copies
  set_assembled_diagonals(m, L);
  L.tiles.clear();
  L.tiles_f32.clear();
  if (dim == 2) {
    build_edge_tiles2(L);
    L.tiles.reserve(L.tiles.size() + (size_t)m->nc * (macro_points(dim, N) / (kTileW * kTileH2) * 2 + 64));
    for (int64_t c = 0; c < m->nc; ++c)
      for (int y0 = 0; y0 <= N; y0 += kTileH2)
        for (int x0 = 0; x0 + y0 <= N; x0 += kTileW) L.tiles.push_back({(int32_t)c, x0, y0, 0});
    while (L.tiles.size() % kWavesPerWG) L.tiles.push_back({-1, 0, 0, 0});
  } else {
    build_tiles3(m, L);
  }
  if (dim == 2) {
    for (int64_t c = 0; c < m->nc; ++c)
      for (int y0 = 0; y0 <= N; y0 += kTileH2F)
        for (int x0 = 0; x0 + y0 <= N; x0 += kTileW) L.tiles_f32.push_back({(int32_t)c, x0, y0, 0});
    while (L.tiles_f32.size() % kWavesPerWG) L.tiles_f32.push_back({-1, 0, 0, 0});
    build_short_tiles2(L, m->nc);
  }

  // row segments of 64 points over every storage point
  L.segs.clear();
  L.segs.reserve((size_t)m->nc * (macro_points(dim, N) / kWave * 2 + 64));
  for (int64_t c = 0; c < m->nc; ++c) {
    const int zmax = dim == 3 ? N : 0;
    for (int z = 0; z <= zmax; ++z) {
      const int M = N - z;
      for (int y = 0; y <= M; ++y)
        for (int x0 = 0; x0 <= M - y; x0 += kWave) L.segs.push_back({(int32_t)c, x0, y, z});
    }
  }
  while (L.segs.size() % kWavesPerWG) L.segs.push_back({-1, 0, 0, 0});
  L.psegs.clear();
  L.psegs.reserve((size_t)m->nc * (macro_points(dim, N) / kWave + (dim == 3 ? N + 2 : 2)) + 64);
  for (int64_t c = 0; c < m->nc; ++c) {
    const int zmax = dim == 3 ? N : 0;
    for (int z = 0; z <= zmax; ++z) {
      const int64_t S = N - z, P = (S + 1) * (S + 2) / 2;
      for (int64_t r0 = 0; r0 < P; r0 += kWave) L.psegs.push_back({(int32_t)c, (int32_t)r0, 0, z});
    }
  }
  while (L.psegs.size() % kWavesPerWG) L.psegs.push_back({-1, 0, 0, 0});
  L.sbase.assign(dim == 3 ? N + 2 : 1, 0);
  if (dim == 3)
    for (int z = 0; z <= N + 1; ++z) L.sbase[z] = (int32_t)slice_base(N, z);
  return MF_OK;
}

namespace {
// Device copies of a level's tables: the small ones share one allocation and
// one copy (one each cost a mesh of ten levels some 250 of both).
struct Upload {
  struct Item {
    void** dst;
    const void* src;
    size_t bytes;
  };
  static constexpr size_t kAlignment = 256, kSmall = 256 * 1024;
  std::vector<Item> items;
  template <class T>
  void add(T** dst, const std::vector<T>& src) {
    *dst = nullptr;
    if (!src.empty()) items.push_back({(void**)dst, src.data(), sizeof(T) * src.size()});
  }
  int run(std::vector<void*>& allocs) {
    auto padded = [](size_t n) { return (n + kAlignment - 1) / kAlignment * kAlignment; };
    auto alloc = [&](size_t bytes, char** out) -> int {
      const hipError_t e = hipMalloc((void**)out, bytes);
      if (e != hipSuccess) return set_error(e == hipErrorOutOfMemory ? MF_ENOMEM : MF_EDEVICE, hipGetErrorString(e));
      allocs.push_back(*out);
      return MF_OK;
    };
    auto copy = [](void* dst, const void* src, size_t bytes) -> int {
      const hipError_t e = hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice);
      return e == hipSuccess ? MF_OK : set_error(MF_EDEVICE, hipGetErrorString(e));
    };
    std::vector<char> small;
    for (const Item& i : items)
      if (i.bytes < kSmall) small.resize(small.size() + padded(i.bytes));
    char* at = nullptr;
    int rc = small.empty() ? MF_OK : alloc(small.size(), &at);
    if (rc) return rc;
    size_t off = 0;
    for (const Item& i : items) {
      char* dst = nullptr;
      if (i.bytes < kSmall) {
        dst = at + off;
        std::memcpy(small.data() + off, i.src, i.bytes);
        off += padded(i.bytes);
      } else {
        if ((rc = alloc(i.bytes, &dst)) || (rc = copy(dst, i.src, i.bytes))) return rc;
      }
      *i.dst = dst;
    }
    return small.empty() ? MF_OK : copy(at, small.data(), small.size());
  }
};
}  // namespace

int upload_level(mf_mesh* m, Level& L) {
  LevelDev& D = L.dev;
  Upload up;
  up.add(&D.md, L.md);
  up.add(&D.tiles, L.tiles);
  up.add(&D.tiles_f32, L.tiles_f32);
  up.add(&D.tiles_short, L.tiles_short);
  up.add(&D.btiles, L.btiles);
  for (int i = 0; i < 2; ++i) up.add(&D.vtiles[i], L.vtiles[i]);
  up.add(&D.faces, L.faces);
  up.add(&D.edges, L.edges);
  up.add(&D.segs, L.segs);
  up.add(&D.psegs, L.psegs);
  up.add(&D.sbase, L.sbase);
  up.add(&D.grp_ptr, L.grp_ptr);
  up.add(&D.copies, L.copies);
  up.add(&D.grp_flag, L.grp_flag);
  up.add(&D.xgrp_ptr, L.xgrp_ptr);
  up.add(&D.cpidx, L.cpidx);
  up.add(&D.xcpidx, L.xcpidx);
  up.add(&D.xgrp_invdiag, L.xgrp_invdiag);
  up.add(&D.own_bits, L.own_bits);
  std::vector<float> f(L.xgrp_invdiag.begin(), L.xgrp_invdiag.end());
  up.add(&D.xgrp_invdiagf, f);
  std::vector<double> zeros(2 * (L.n_partials() + 1), 0.0);
  up.add(&D.part, zeros);
  std::vector<double> z2(2, 0.0);
  up.add(&D.result, z2);
  (void)m;
  return up.run(D.allocs);
}

// ---------------------------------------------------------------- coarse direct solve
// Dense inverse of the assembled interior block at a coarse level, summed
// from the same element matrices the kernels use.
int build_coarse_solver(mf_mesh* m, int level) {
  Level& L = m->levels[level];
  if (L.ncoarse > 0 || !L.cfirst.empty()) return MF_OK;
  const int dim = m->dim, d1 = dim + 1;
  const int N = L.N;
  const ElemTable ET = elem_table(dim);
  // unique ids of all storage points by key
  struct Ent {
    PointKey k;
    int64_t sidx;
    int32_t macro, x, y, z;
  };
  std::vector<Ent> ent;
  for (int64_t c = 0; c < m->nc; ++c) {
    const int zmax = dim == 3 ? N : 0;
    for (int z = 0; z <= zmax; ++z)
      for (int y = 0; y <= N - z; ++y)
        for (int x = 0; x <= N - z - y; ++x) {
          const int64_t s = L.base[c] + (dim == 2 ? idx2(N, x, y) : idx3(N, x, y, z));
          ent.push_back({point_key(dim, &m->cells[c * d1], N, x, y, z), s, (int32_t)c, x, y, z});
        }
  }
  std::sort(ent.begin(), ent.end(), [](const Ent& a, const Ent& b) {
    if (!(a.k == b.k)) return a.k < b.k;
    return a.sidx < b.sidx;
  });
  std::vector<int64_t> uid_of(L.storage, -1);
  std::vector<int64_t> unk_of_uid;  // -1 for Dirichlet
  int64_t nu = 0, nunk = 0;
  L.cfirst.clear();
  L.cptr.clear();
  L.cidx.clear();
  std::vector<std::vector<int64_t>> copies_of_unk;
  for (size_t i = 0; i < ent.size(); ++i) {
    if (i == 0 || !(ent[i].k == ent[i - 1].k)) {
      const int s = support_mask(dim, N, ent[i].x, ent[i].y, ent[i].z);
      const bool dir = (m->dir_mask[ent[i].macro] >> s) & 1;
      unk_of_uid.push_back(dir ? -1 : nunk);
      if (!dir) {
        copies_of_unk.emplace_back();
        ++nunk;
      }
      ++nu;
    }
    uid_of[ent[i].sidx] = nu - 1;
    const int64_t k = unk_of_uid[nu - 1];
    if (k >= 0) copies_of_unk[k].push_back(ent[i].sidx);
  }
  if (nunk > 4096) return set_error(MF_ENOTSUP, "coarse level has more than 4096 unknowns; choose a coarser level");
  std::vector<double> A((size_t)nunk * nunk, 0.0);
  for (int64_t c = 0; c < m->nc; ++c) {
    const MacroDev& M = L.md[c];
    const int zmax = dim == 3 ? N : 0;
    for (int az = 0; az <= zmax; ++az)
      for (int ay = 0; ay <= N; ++ay)
        for (int ax = 0; ax <= N; ++ax)
          for (int t = 0; t < ET.ntypes; ++t) {
            if (ax + ay + az > N - ET.slack[t]) continue;
            int64_t ids[4];
            for (int v = 0; v < ET.nv; ++v) {
              const int x = ax + ET.off[t][v][0], y = ay + ET.off[t][v][1], z = az + ET.off[t][v][2];
              const int64_t s = L.base[c] + (dim == 2 ? idx2(N, x, y) : idx3(N, x, y, z));
              ids[v] = unk_of_uid[uid_of[s]];
            }
            for (int v = 0; v < ET.nv; ++v)
              for (int u = 0; u < ET.nv; ++u)
                if (ids[v] >= 0 && ids[u] >= 0) A[ids[v] * nunk + ids[u]] += M.K[t][v * 4 + u];
          }
  }
  // Cholesky A = C C^T, then A^{-1} = C^{-T} C^{-1}
  const int64_t n = nunk;
  std::vector<double> C(A);
  for (int64_t j = 0; j < n; ++j) {
    double d = C[j * n + j];
    for (int64_t k = 0; k < j; ++k) d -= C[j * n + k] * C[j * n + k];
    if (!(d > 0.0)) return set_error(MF_ENUMERIC, "coarse operator is not positive definite");
    d = std::sqrt(d);
    C[j * n + j] = d;
    for (int64_t i = j + 1; i < n; ++i) {
      double s = C[i * n + j];
      for (int64_t k = 0; k < j; ++k) s -= C[i * n + k] * C[j * n + k];
      C[i * n + j] = s / d;
    }
  }
  std::vector<double> Ci((size_t)n * n, 0.0);  // C^{-1}, lower triangular
  for (int64_t col = 0; col < n; ++col)
    for (int64_t i = col; i < n; ++i) {
      double s = (i == col) ? 1.0 : 0.0;
      for (int64_t k = col; k < i; ++k) s -= C[i * n + k] * Ci[k * n + col];
      Ci[i * n + col] = s / C[i * n + i];
    }
  L.cinv.assign((size_t)n * n, 0.0);
  for (int64_t i = 0; i < n; ++i)
    for (int64_t j = 0; j < n; ++j) {
      double s = 0.0;
      for (int64_t k = std::max(i, j); k < n; ++k) s += Ci[k * n + i] * Ci[k * n + j];
      L.cinv[i * n + j] = s;
    }
  L.cptr.push_back(0);
  for (int64_t k = 0; k < n; ++k) {
    L.cfirst.push_back((int32_t)copies_of_unk[k][0]);
    for (int64_t s : copies_of_unk[k]) L.cidx.push_back(s);
    L.cptr.push_back((int32_t)L.cidx.size());
  }
  L.ncoarse = n;
  if (m->host_only) return MF_OK;
  int rc;
  if ((rc = dev_upload(&L.dev.cinv, L.cinv))) return rc;
  std::vector<float> f(L.cinv.begin(), L.cinv.end());
  if ((rc = dev_upload(&L.dev.cinvf, f))) return rc;
  if ((rc = dev_upload(&L.dev.cfirst, L.cfirst))) return rc;
  if ((rc = dev_upload(&L.dev.cptr, L.cptr))) return rc;
  if ((rc = dev_upload(&L.dev.cidx, L.cidx))) return rc;
  return MF_OK;
}

// ---------------------------------------------------------------- whole mesh
int build_mesh(mf_mesh* m) {
  const int dim = m->dim, d1 = dim + 1;
  for (int64_t i = 0; i < m->nc * d1; ++i)
    if (m->cells[i] < 0 || m->cells[i] >= m->nv) return set_error(MF_EINVAL, "cell vertex id out of range");
  for (int64_t c = 0; c < m->nc; ++c) {
    const double* P0 = &m->coords[m->cells[c * d1] * dim];
    double J[3][3] = {{0}}, scale = 0.0;
    for (int k = 1; k <= dim; ++k)
      for (int r = 0; r < dim; ++r) {
        J[r][k - 1] = m->coords[m->cells[c * d1 + k] * dim + r] - P0[r];
        scale = std::max(scale, std::fabs(J[r][k - 1]));
      }
    double det = dim == 2 ? J[0][0] * J[1][1] - J[0][1] * J[1][0]
                          : J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
                                J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                                J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
    if (!(std::fabs(det) > 1e-14 * std::pow(scale, dim)))
      return set_error(MF_EINVAL, "degenerate macro cell " + std::to_string(c));
  }
  int rc = build_topology(m);
  if (rc) return rc;
  m->levels.resize(m->max_level + 1);
  for (int l = 0; l <= m->max_level; ++l)
    if ((rc = build_level(m, l, m->levels[l]))) return rc;
  if (!m->host_only) {
    hipError_t e = hipGetDevice(&m->device);
    if (e != hipSuccess) return set_error(MF_EDEVICE, hipGetErrorString(e));
    for (int l = 0; l <= m->max_level; ++l)
      if ((rc = upload_level(m, m->levels[l]))) return rc;
  }
  return build_2d_tables(m);
}

void free_device(mf_mesh* m) {
  for (auto& L : m->levels) {
    LevelDev& D = L.dev;
    for (void* p : D.allocs) (void)hipFree(p);
    void* ptrs[] = {D.cinv, D.cinvf, D.cfirst, D.cptr, D.cidx, D.p2_tiles};
    for (void* p : ptrs)
      if (p) (void)hipFree(p);
    D = LevelDev{};
  }
  if (m->p2_dev) (void)hipFree(m->p2_dev);
  m->p2_dev = nullptr;
  if (m->geo2_dev) (void)hipFree(m->geo2_dev);
  m->geo2_dev = nullptr;
}

void storage_keys(const mf_mesh* m, int level, int64_t* vids, int32_t* wts) {
  const Level& L = m->levels[level];
  const int dim = m->dim, d1 = dim + 1;
  const int N = L.N;
  for (int64_t c = 0; c < m->nc; ++c) {
    const int zmax = dim == 3 ? N : 0;
    for (int z = 0; z <= zmax; ++z)
      for (int y = 0; y <= N - z; ++y)
        for (int x = 0; x <= N - z - y; ++x) {
          const int64_t s = L.base[c] + (dim == 2 ? idx2(N, x, y) : idx3(N, x, y, z));
          const PointKey k = point_key(dim, &m->cells[c * d1], N, x, y, z);
          for (int i = 0; i < d1; ++i) {
            vids[s * d1 + i] = k.v[i];
            wts[s * d1 + i] = k.w[i];
          }
        }
  }
}

}  // namespace mf

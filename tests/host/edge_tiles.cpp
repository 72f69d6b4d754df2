// The tiles of shared DoFs that mesh set-up makes, for meshes read from stdin
// ("dim level vertices cells", coordinates, cells): in every list that holds them
// each copy lies in exactly one tile, the copies of a DoF in consecutive lanes
// from its head, and the DoFs are those of the group lists.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "mesh.hpp"
#include "mf_stencil.h"

using namespace mf;

static void check(bool ok, const char* what, const Level& L) {
  if (ok) return;
  printf("FAIL %s at level %d\n", what, L.level);
  exit(1);
}

// group[i]: the DoF of copy i of Level::edges
static void check_list(const Level& L, const std::vector<Tile>& tiles, size_t n, int steps, const std::vector<int>& group,
                       const std::vector<int>& size) {
  std::vector<int> seen(L.edges.size(), 0);
  for (size_t t = 0; t < n; ++t) {
    const Tile& T = tiles[t];
    if (T.macro != kEdgeTile && T.macro != kEdgeBigTile) continue;
    check(T.x0 >= 0 && T.y0 > 0 && T.x0 + T.y0 + T.z <= (int)L.edges.size(), "tile bounds", L);
    check(T.z == 0 || (steps == 2 && T.macro == kEdgeTile), "second step", L);
    const bool big = T.macro == kEdgeBigTile;
    check(big == (size[group[T.x0]] > kWave) && (!big || T.y0 == size[group[T.x0]]), "tile of one DoF", L);
    for (int s = 0, at = T.x0; s < 2; at += T.y0, ++s) {
      const int m = s == 0 ? T.y0 : T.z;
      check(big || m <= kWave, "lanes", L);
      for (int i = 0; i < m; ++i) {
        const EdgeCopy& e = L.edges[at + i];
        ++seen[at + i];
        check(big ? group[at + i] == group[T.x0] : e.copies == size[group[at + i]], "copies", L);
        if (big) continue;
        check(e.head <= i && i < e.head + e.copies && e.head + e.copies <= m, "head", L);
        check(group[at + e.head] == group[at + i] && group[at + e.head + e.copies - 1] == group[at + i], "lanes of a DoF", L);
      }
    }
  }
  for (int s : seen) check(s == 1, "a copy in one tile", L);
}

int main() {
  int dim, level;
  long nv, nc;
  while (scanf("%d %d %ld %ld", &dim, &level, &nv, &nc) == 4) {
    std::vector<double> co(nv * dim);
    std::vector<int64_t> ce(nc * (dim + 1));
    for (double& v : co)
      if (scanf("%lf", &v) != 1) return 2;
    for (int64_t& v : ce) {
      long q;
      if (scanf("%ld", &q) != 1) return 2;
      v = q;
    }
    for (int flags : {0, (int)MF_FLAG_DIRICHLET}) {
      mf_mesh* m = nullptr;
      if (create_macro_mesh(dim, nv, co.data(), nc, ce.data(), level, flags | MF_FLAG_HOST_ONLY, &m)) return 3;
      for (const Level& L : m->levels) {
        // the DoFs, in order, that the tiles must hold
        std::vector<int> group, size;
        std::vector<int64_t> idx;
        std::vector<bool> fixed;
        auto add = [&](const std::vector<int32_t>& ptr, int64_t g, const std::vector<int64_t>& at, bool dirichlet) {
          for (int c = ptr[g]; c < ptr[g + 1]; ++c) {
            group.push_back((int)size.size());
            idx.push_back(at[c]);
            fixed.push_back(dirichlet);
          }
          size.push_back(ptr[g + 1] - ptr[g]);
        };
        if (dim == 2) {
          for (int64_t g = 0; g < L.nxgroups(); ++g) add(L.xgrp_ptr, g, L.xcpidx, false);
        } else {
          for (int64_t g = 0; g < L.ngroups(); ++g) {
            const Copy& k = L.copies[L.grp_ptr[g]];
            const int mask = support_mask(3, L.N, k.x, k.y, k.z);
            const bool face = __builtin_popcount(mask) == 3, dirichlet = L.grp_flag[g] & 1;
            if ((face && L.N >= kMinFaceN) || ((mask == 13 || mask == 14) && dirichlet)) continue;
            add(L.grp_ptr, g, L.cpidx, dirichlet);
          }
        }
        check(L.edges.size() == idx.size(), "number of copies", L);
        for (size_t i = 0; i < idx.size(); ++i) {
          const EdgeCopy& e = L.edges[i];
          const int64_t at = L.base[e.macro] + (dim == 2 ? idx2(L.N, e.x, e.y) : idx3(L.N, e.x, e.y, e.z));
          check(e.idx == idx[i] && at == idx[i], "storage index", L);
          check(e.mask == support_mask(dim, L.N, e.x, e.y, e.z) && (e.dirichlet != 0) == fixed[i], "copy", L);
        }
        check_list(L, L.tiles, L.tiles.size(), dim == 2 ? 2 : 1, group, size);
        check_list(L, L.btiles, L.btiles.size(), dim == 2 ? 2 : 1, group, size);
        if (dim == 3) continue;
        check_list(L, L.tiles, (size_t)L.ewgs * kWavesPerWG, 2, group, size);
        check_list(L, L.tiles_f32, (size_t)L.ewgs * kWavesPerWG, 2, group, size);
        if (L.short_rows) check_list(L, L.tiles_short, (size_t)L.ewgs_short * kWavesPerWG, 1, group, size);
      }
      destroy_macro_mesh(m);
    }
  }
  printf("OK\n");
  return 0;
}

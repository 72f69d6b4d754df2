// Tile shapes of the stencil launches: levels of meshes read from stdin ("dim
// level vertices cells", coordinates, cells) take shapes that have a kernel, with
// lists of that shape, and a launch of a shape that has none is an error.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "launch.hpp"
#include "mesh.hpp"
#include "mf_stencil.h"

using namespace mf;

static void check(bool ok, const char* what, int a, int b) {
  if (ok) return;
  printf("FAIL %s: %d %d\n", what, a, b);
  exit(1);
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
    mf_mesh* m = nullptr;
    if (create_macro_mesh(dim, nv, co.data(), nc, ce.data(), level, MF_FLAG_DIRICHLET | MF_FLAG_HOST_ONLY, &m)) return 3;
    for (const Level& L : m->levels) {
      if (dim == 3) {
        check(shape3(L.N).R >= 1 && shape3(L.N).R <= kMaxR3, "rows per band", L.level, shape3(L.N).R);
        continue;
      }
      for (int dtype : {(int)MF_F64, (int)MF_F32}) {
        const int rows = L.rows2(dtype);
        check(rows == kTileShort[0] || rows == kTileShort[1] || rows == kTileH2 || (dtype == MF_F32 && rows == kTileH2F),
              "rows per tile", L.level, rows);
        int64_t covered = 0;
        for (const Tile& t : L.tiles_for(dtype)) {
          if (t.macro < 0) continue;
          check(t.y0 % rows == 0 && t.x0 % kTileW == 0, "tile", t.x0, t.y0);
          for (int y = t.y0; y < t.y0 + rows && t.x0 + y <= L.N; ++y)
            covered += std::min(kTileW, L.N + 1 - t.x0 - y);
        }
        check(covered == L.storage, "points covered", L.level, dtype);
      }
    }
    destroy_macro_mesh(m);
  }
  for (int dim2 : {2, 3})
    for (int dtype : {(int)MF_F64, (int)MF_F32})
      for (int variant : {0, 5, 7, 16, 32}) {
        if (dim2 == 2 && dtype == MF_F32 && variant == kTileH2F) continue;
        BatchOp op{};
        op.kind = kOpStencil;
        op.dtype = dtype;
        op.dim = dim2;
        op.mode = kApply;
        op.nseg = op.nwg = 1;
        op.variant = variant;
        check(launch_stencil_batch(op, nullptr, nullptr) == MF_EINVAL, "a shape without a kernel", dim2, variant);
      }
  printf("OK\n");
  return 0;
}

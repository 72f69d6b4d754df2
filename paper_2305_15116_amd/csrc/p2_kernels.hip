// Fused P2 operator for 2D macro meshes (gfx950): y = A x over the vertex
// and edge-midpoint DoFs in one pass (the paper's four P2 kernels,
// Performance Modeling section, fused as its Conclusion proposes).
//
// Interior DoFs: a 64-lane wavefront walks fine rows upward.  Lane i holds
// the fine columns xa = x0 - 2 + 2i (even) and xa + 1 of each row, so in an
// even row it computes a vertex row (19 neighbours) and a horizontal-edge row
// (9), in an odd row a vertical- and a diagonal-edge row (9 each).  Every
// neighbour is at most two columns and two rows away, i.e. in the lane itself
// or in lanes i +- 1 (DPP shifts), and in the five rows kept in registers, so
// each source value is read from memory once per tile.  Opposite neighbours
// share a weight (p2.hpp) and are added before the multiply.
//
// Macro-boundary DoFs (about 3 * 2^(l+1) per macro) have workgroups of their own
// at the head of the launch: a lane sums the element-matrix rows of the
// micro-triangles of its macro that contain its point.  DoFs shared by macros
// take a lane per copy and sum these over the copies; Dirichlet ones copy x.
//
// Bound: memory (x read, y written).  Against a launch each for the interior, the
// boundary and the sums over shared DoFs: five triangles at level 11 FP64 157.8 ->
// 149.4 us (4.5 TB/s), FP32 90.2 -> 84.5; seven at level 7 12.8 -> 6.4, 11.4 -> 5.9.
// Fewer workgroups at once (5, 4, 3 per CU) are slower: 149, 157, 179 us.

#include <hip/hip_runtime.h>

#include "edges.hpp"
#include "launch.hpp"
#include "p2.hpp"
#include "wave.hpp"

namespace mf {

namespace {

using wave::dn1;
using wave::up1;

template <typename T>
struct P2Tab;
template <>
struct P2Tab<double> {
  static __device__ __forceinline__ const double* w(const P2Macro& P) { return P.w; }
  static __device__ __forceinline__ const double* K(const P2Macro& P) { return P.K; }
};
template <>
struct P2Tab<float> {
  static __device__ __forceinline__ const float* w(const P2Macro& P) { return P.wf; }
  static __device__ __forceinline__ const float* K(const P2Macro& P) { return P.Kf; }
};

// One fine row as a lane sees it: its even column a, the odd column b after
// it, and the shifted copies the stencils use (ua: a of lane - 1, i.e. column
// xa - 2; da: a of lane + 1, column xa + 2; ub: b of lane - 1, column xa - 1).
template <typename T>
struct Row {
  T a, b, ua, da, ub;
};
template <typename T>
__device__ __forceinline__ Row<T> row_of(T a, T b) {
  return Row<T>{a, b, up1(a), dn1(a), up1(b)};
}

// Two adjacent entries, loaded or stored as one 16-byte (FP64) access; rows
// start at any entry, so only the element alignment is assumed (gfx950
// global memory accesses need dword alignment only).
template <typename T>
struct Pair;
template <>
struct Pair<double> {
  typedef double V __attribute__((ext_vector_type(2), aligned(8)));
};
template <>
struct Pair<float> {
  typedef float V __attribute__((ext_vector_type(2), aligned(4)));
};

// Columns xa and xa + 1 of row r of the fine triangle (side M), with the row
// clamped to [0, last] and the columns into the row: a valid point for every
// lane (clamped values only feed halo lanes and points that are not stored).
template <typename T>
__device__ __forceinline__ void ld_pair(const T* __restrict__ X, int M, int r, int last, int xa, T& a, T& b) {
  const int rr = min(max(r, 0), last);
  const int S = M - rr;
  const T* row = X + row_start(M, rr);
  if (sizeof(T) == 4) {
    // FP32: two 4-byte loads measured faster than one 8-byte pair load
    a = row[min(max(xa, 0), S)];
    b = row[min(max(xa + 1, 0), S)];
  } else if (S >= 1) {
    // one 2-element load at a start kept inside the row; a lane past the row
    // end takes the last element, a lane before its start the first
    const int st = min(max(xa, 0), S - 1);
    const typename Pair<T>::V v = *(const typename Pair<T>::V*)(row + st);
    a = xa >= S ? v.y : v.x;
    b = xa < 0 ? v.x : v.y;
  } else {
    a = row[0];
    b = a;
  }
}

constexpr int kP2U = 4;  // rows loaded ahead
static_assert(kP2H % 2 == 0 && kP2H >= kP2U, "tile height");

template <typename T>
__device__ __forceinline__ void p2_tile(int x0, int y0, const MacroDev& Md, const P2Macro& P, const T* __restrict__ X,
                                        T* __restrict__ Y) {
  const int lane = threadIdx.x & (kWave - 1);
  const int M = Md.N;  // fine side
  const int xa = x0 - 2 + 2 * lane;
  const bool lane_out = lane >= 1 && lane <= kTileW;
  const int nrows = min(kP2H, M - y0);  // rows that can hold interior points (Y <= M - 1)
  const int last = min(y0 + nrows + 1, M);
  X += Md.base;
  Y += Md.base;
  const T* w = P2Tab<T>::w(P);
  T wt[kP2Weights];
#pragma unroll
  for (int k = 0; k < kP2Weights; ++k) wt[k] = w[k];

  Row<T> r0, r1, r2, r3;  // rows Y-2 .. Y+1 of the current output row Y
  {
    T a, b;
    ld_pair(X, M, y0 - 2, last, xa, a, b);
    r0 = row_of(a, b);
    ld_pair(X, M, y0 - 1, last, xa, a, b);
    r1 = row_of(a, b);
    ld_pair(X, M, y0, last, xa, a, b);
    r2 = row_of(a, b);
    ld_pair(X, M, y0 + 1, last, xa, a, b);
    r3 = row_of(a, b);
  }
  T qa[kP2U], qb[kP2U];  // raw rows y0+2 .. loaded ahead
#pragma unroll
  for (int k = 0; k < kP2U; ++k) ld_pair(X, M, y0 + 2 + k, last, xa, qa[k], qb[k]);

#pragma unroll
  for (int k = 0; k < kP2H; ++k) {
    const Row<T> r4 = row_of(qa[k % kP2U], qb[k % kP2U]);  // row Y+2
    if (k + kP2U + 1 <= kP2H) ld_pair(X, M, y0 + 2 + k + kP2U, last, xa, qa[k % kP2U], qb[k % kP2U]);
    if (k < nrows) {
      const int yy = y0 + k;
      T oa, ob;
      if ((k & 1) == 0) {
        // vertex at xa, horizontal edge at xa + 1
        oa = wt[0] * r2.a;
        oa = fma(wt[1], r2.da + r2.ua, oa);
        oa = fma(wt[2], r4.a + r0.a, oa);
        oa = fma(wt[3], r0.da + r4.ua, oa);
        oa = fma(wt[4], r2.b + r2.ub, oa);
        oa = fma(wt[5], r3.a + r1.a, oa);
        oa = fma(wt[6], r1.b + r3.ub, oa);
        oa = fma(wt[7], r3.b + r1.ub, oa);
        oa = fma(wt[8], r1.da + r3.ua, oa);
        oa = fma(wt[9], r0.b + r4.ub, oa);
        ob = wt[10] * r2.b;
        ob = fma(wt[11], r2.da + r2.a, ob);
        ob = fma(wt[12], r3.b + r1.b, ob);
        ob = fma(wt[13], r3.a + r1.da, ob);
        ob = fma(wt[14], r4.a + r0.da, ob);
      } else {
        // vertical edge at xa, diagonal edge at xa + 1
        oa = wt[15] * r2.a;
        oa = fma(wt[16], r3.a + r1.a, oa);
        oa = fma(wt[17], r1.da + r3.ua, oa);
        oa = fma(wt[18], r1.b + r3.ub, oa);
        oa = fma(wt[19], r2.b + r2.ub, oa);
        ob = wt[20] * r2.b;
        ob = fma(wt[21], r3.da + r1.a, ob);
        ob = fma(wt[22], r1.da + r3.a, ob);
        ob = fma(wt[23], r3.b + r1.b, ob);
        ob = fma(wt[24], r2.da + r2.a, ob);
      }
      // interior points only: X >= 1, Y >= 1, X + Y <= M - 1
      T* yrow = Y + row_start(M, yy);
      const bool va = lane_out && yy >= 1 && xa >= 1 && xa + yy <= M - 1;
      const bool vb = lane_out && yy >= 1 && xa + 1 + yy <= M - 1;
      if (va && vb) {
        typename Pair<T>::V v;
        v.x = oa;
        v.y = ob;
        *(typename Pair<T>::V*)(yrow + xa) = v;
      } else {
        if (va) yrow[xa] = oa;
        if (vb) yrow[xa + 1] = ob;
      }
    }
    r0 = r1;
    r1 = r2;
    r2 = r3;
    r3 = r4;
  }
}

// Row of macro-boundary point (x, y) from the micro-triangles of its macro:
// triangle (a, b, up / down) has its points at 2 (a, b) + the offsets below.
template <typename T>
__device__ __forceinline__ T p2_partial(const MacroDev& Md, const P2Macro& P, const T* __restrict__ X, int x, int y) {
  constexpr int kX[2][6] = {{2, 0, 2, 1, 1, 2}, {0, 2, 0, 1, 1, 0}}, kY[2][6] = {{2, 2, 0, 2, 1, 1}, {0, 0, 2, 0, 1, 1}};
  const T* K = P2Tab<T>::K(P);
  const int M = Md.N, nc = M / 2;
  X += Md.base;
  T acc = T(0);
#pragma unroll
  for (int up = 1; up >= 0; --up)
#pragma unroll
    for (int db = -1; db <= 0; ++db)
#pragma unroll
      for (int da = -1; da <= 0; ++da) {
        const int a = (x >> 1) + da, b = (y >> 1) + db;
        int row = -1;  // the point's in the triangle
#pragma unroll
        for (int q = 0; q < 6; ++q)
          if (x - 2 * a == kX[up][q] && y - 2 * b == kY[up][q]) row = q;
        if (row < 0 || a < 0 || b < 0 || a + b > nc - 1 - (up ? 0 : 1)) continue;
#pragma unroll
        for (int q = 0; q < 6; ++q)
          acc = fma(K[row * 6 + q], X[idx2(M, 2 * a + kX[up][q], 2 * b + kY[up][q])], acc);
      }
  return acc;
}

template <typename T>
struct P2Args {
  const Tile* edges_at;  // tiles of shared DoFs (ewg workgroups)
  const EdgeCopy* edges;
  const Tile* tiles;     // interior tiles
  int ewg, bwg, nwg;     // workgroups of shared DoFs, of other boundary DoFs, of all
  int nmacro, M;
  const MacroDev* md;
  const P2Macro* p2;
  const T* X;
  T* Y;
};

// Macro-boundary DoF k of macro c that is its macro's alone or Dirichlet: k in
// [0, M] on y = 0, (M, 2M] on x = 0 (y = k - M), (2M, 3M) on the far edge x + y = M
// (y = k - 2M).
template <typename T>
__device__ __forceinline__ void p2_boundary(const P2Args<T>& a, int64_t t) {
  const int M = a.M, per = 3 * M;
  if (t >= (int64_t)a.nmacro * per) return;
  const int c = (int)(t / per), k = (int)(t % per);
  const int y = k <= M ? 0 : (k <= 2 * M ? k - M : k - 2 * M), x = k <= M ? k : (k <= 2 * M ? 0 : M - y);
  const MacroDev& Md = a.md[c];
  const int mask = support_mask(2, M, x, y, 0);
  const bool dir = (Md.dir_mask >> mask) & 1;
  if (!dir && ((Md.shared_mask >> mask) & 1)) return;
  const int64_t i = Md.base + idx2(M, x, y);
  a.Y[i] = dir ? a.X[i] : p2_partial<T>(Md, a.p2[c], a.X, x, y);
}

template <typename T>
__global__ __launch_bounds__(kWG) void p2_kernel(const P2Args<T> a) {
  int g = wave::xcd_wg_lead(a.nwg, a.ewg, a.bwg, wave::kRuns2);
  if (g < 0) return;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (g < a.ewg) {
    const Tile t = load_seg(a.edges_at, g * kWavesPerWG + wv);
    if (t.macro != -1)
      shared_rows(a.edges, t, a.Y, [&](const EdgeCopy& e) { return p2_partial<T>(a.md[e.macro], a.p2[e.macro], a.X, e.x, e.y); });
    return;
  }
  g -= a.ewg;
  if (g < a.bwg) return p2_boundary<T>(a, (int64_t)g * kWG + threadIdx.x);
  const Tile t = load_seg(a.tiles, (g - a.bwg) * kWavesPerWG + wv);
  if (t.macro < 0) return;
  p2_tile<T>(t.x0, t.y0, a.md[t.macro], a.p2[t.macro], a.X, a.Y);
}

template <typename T>
int run_p2(const mf_mesh* m, const Level& F, const void* x, void* y, hipStream_t s) {
  const int64_t nb = (int64_t)m->nc * 3 * F.N;
  const int bwg = (int)((nb + kWG - 1) / kWG), nwg = F.ewgs + bwg + (int)(F.p2_tiles.size() / kWavesPerWG);
  const P2Args<T> a{F.dev.tiles, F.dev.edges, F.dev.p2_tiles, F.ewgs, bwg,        nwg,  (int)m->nc,
                    F.N,         F.dev.md,    m->p2_dev,      (const T*)x, (T*)y};
  hipLaunchKernelGGL(p2_kernel<T>, dim3(wave::xcd_grid(nwg, F.ewgs, bwg, wave::kRuns2)), dim3(kWG), 0, s, a);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? MF_OK : set_error(MF_EDEVICE, hipGetErrorString(e));
}

}  // namespace

int launch_p2_apply(const mf_mesh* m, int level, int dtype, const void* x, void* y, hipStream_t s) {
  const Level& F = m->levels[level + 1];
  return dtype == MF_F64 ? run_p2<double>(m, F, x, y, s) : run_p2<float>(m, F, x, y, s);
}

}  // namespace mf

// Device code of the macro edges and vertices (gfx950; in 2D the edges shared by
// macros): rows summed over all copies of a DoF within one launch.
#pragma once

#include <hip/hip_runtime.h>

#include "rows.hpp"

namespace mf {

// Row value of a DoF that is not Dirichlet, from its assembled sum acc; inv = 1
// / assembled diagonal (Jacobi).
template <typename T, int MODE>
__device__ __forceinline__ T row_value(T acc, T xc, T bv, T omega, T inv) {
  if (MODE == kApply || MODE == kApplyDot) return acc;
  if (MODE == kJacobi || MODE == kJacobi2) return fma(omega * inv, bv - acc, xc);
  if (MODE == kResidual) return bv - acc;
  return bv;
}
template <typename T, int MODE>
__device__ __forceinline__ T dirichlet_row(T xc, T bv) {
  if (MODE == kJacobi2) return T(0);
  return MODE == kResidual ? bv - xc : (MODE == kNormB ? bv : xc);
}

// The iterate at a point with support `mask` whose stored value is v: v, or
// (kJacobi2, whose X is b) the first sweep's omega D^-1 b.
template <typename T, int MODE>
__device__ __forceinline__ T iterate(const MacroDev& M, int mask, T omega, T v) {
  return MODE == kJacobi2 ? (omega * Prec<T>::zinv(M, mask)) * v : v;
}

// The 2D stencil neighbours of point (x, y) of a macro of side N, stored at X
// (table order): neighbours along x in pairs (8 or 16 bytes), four accesses
// instead of seven, since the copies of an edge lie a row apart and each access
// takes a cycle per lane.  Rows and points outside the macro read others of its
// points, and their values are some point's: the caller drops them.
template <typename T>
__device__ __forceinline__ void neighbours2(const T* X, int N, int x, int y, T (&v)[7]) {
  typedef T Pair __attribute__((ext_vector_type(2), aligned(sizeof(T))));
  const bool x0 = x == 0, y0 = y == 0, far = x + y == N, first = x0 && !far;  // first: its row's, with a successor
  const int l = N + 1 - y;                                                     // the row's length
  const int at = first ? 0 : -1;
  const Pair m = *(const Pair*)(X + at);                                     // first: C, E; else W, C
  const Pair s = *(const Pair*)(X + (y0 ? at : -l - 1));                     // S, SE
  const Pair n = *(const Pair*)(X + (far ? (x0 ? at : l - 2) : l - 1));      // NW, N; far: its predecessor, NW
  const T e = X[far ? 0 : 1];
  v[0] = s.x, v[1] = s.y, v[2] = m.x, v[3] = first ? m.x : m.y, v[4] = e, v[5] = far ? n.y : n.x, v[6] = n.y;
}

// Partial row of one copy of a macro edge or vertex DoF: the partial stencil
// of its support mask, neighbours outside the macro dropped, table order.  xc:
// the iterate at the copy.
template <typename T, int DIM, int MODE>
__device__ __forceinline__ T copy_partial(const MacroDev* md, const EdgeCopy& k, const T* X, T omega, T& xc) {
  constexpr StencilTable ST = stencil_table(DIM);
  const MacroDev& M = md[k.macro];
  const int N = M.N;
  T v[ST.n];
  if constexpr (DIM == 3) {
    int off[15];
    nbr_offsets3(N, k.y, k.z, off);
#pragma unroll
    for (int o = 0; o < ST.n; ++o) {
      const int nx = k.x + ST.off[o][0], ny = k.y + ST.off[o][1], nz = k.z + ST.off[o][2];
      v[o] = X[nx >= 0 && ny >= 0 && nz >= 0 && nx + ny + nz <= N ? k.idx + off[o] : k.idx];
    }
  } else {
    neighbours2(X + k.idx, N, k.x, k.y, v);
  }
  T p = T(0);
#pragma unroll
  for (int o = 0; o < ST.n; ++o) {
    const int nx = k.x + ST.off[o][0], ny = k.y + ST.off[o][1], nz = k.z + ST.off[o][2];
    const bool in = nx >= 0 && ny >= 0 && nz >= 0 && nx + ny + nz <= N;
    const T vo = iterate<T, MODE>(M, support_mask(DIM, N, nx, ny, nz), omega, v[o]);
    p = fma(Prec<T>::w(M, k.mask, o), in ? vo : T(0), p);
    if (o == ST.centre) xc = vo;
  }
  return p;
}

// Copies of macro edge and vertex DoFs, one per lane; the copies of a DoF sit in
// consecutive lanes from its head (kEdgeTile: t.y0 copies, then t.z in a second
// step), or, with more than 64 copies, one DoF fills the tile in steps of 64
// (kEdgeBigTile).  The copies' partial rows are summed in list order by every
// lane of the DoF.
//
// Bound: latency.  In 2D this replaces a launch after every pass that summed
// the partial rows that the walk wrote: seven triangles at level 8, FP64 apply / Jacobi
// / residual 8.7 / 9.6 / 9.5 -> 5.1 / 5.9 / 5.6 us, FP32 10.6 / 11.8 / 11.9 -> 7.0 / 7.6 / 7.7;
// two at level 12 FP32 39.5 / 49.5 / 51.9 -> 33.3 / 43.2 / 45.5.  Meshes of many
// macros: the accesses, each lane's on a line of its own.  With 2D neighbours one by
// one, x twice, b at every copy and 40-byte records, 3,200 triangles at level 7
// took 176 us instead of 166 per FP64 apply, 512 at level 6 20.3 instead of 14.9.
template <typename T, int DIM, int MODE>
__device__ __forceinline__ void edge_rows(const StencilArgs<T>& a, const Tile& t, double& ss, double& mx) {
  constexpr bool kX = MODE != kNormB;
  constexpr bool kB = MODE != kApply && MODE != kApplyDot;
  const int lane = threadIdx.x & (kWave - 1);
  const EdgeCopy* L = a.edges + t.x0;
  // (2D: the exchange list, without Dirichlet DoFs)
  auto fixed = [](const EdgeCopy& k) { return DIM == 3 && k.dirichlet; };
  // a copy's partial row p, x and b (b of the heads, and of Dirichlet copies)
  auto load = [&](const EdgeCopy& k, bool live, bool head, T& p, T& xo, T& bo) {
    p = xo = bo = T(0);
    if (kB && live && (head || fixed(k))) bo = a.B[k.idx];
    if (kX && live && fixed(k)) xo = iterate<T, MODE>(a.md[k.macro], k.mask, a.omega, a.X[k.idx]);
    if (kX && live && !fixed(k)) p = copy_partial<T, DIM, MODE>(a.md, k, a.X, a.omega, xo);
  };
  auto inverse = [&](const EdgeCopy& k) {
    return MODE == kJacobi || MODE == kJacobi2 ? Prec<T>::zinv(a.md[k.macro], k.mask) : T(0);
  };
  if (t.macro == kEdgeBigTile) {
    T acc = T(0), xh = T(0), bh = T(0);
    for (int c0 = 0; c0 < t.y0; c0 += kWave) {
      const int n = min(kWave, t.y0 - c0);
      T p, xo, bo;
      load(L[c0 + min(lane, n - 1)], lane < n, c0 == 0 && lane == 0, p, xo, bo);
      if (c0 == 0) xh = __shfl(xo, 0, kWave), bh = __shfl(bo, 0, kWave);
      if (fixed(L[0])) break;
      for (int i = 0; kX && i < n; ++i) acc += __shfl(p, i, kWave);
    }
    const T out = fixed(L[0]) ? dirichlet_row<T, MODE>(xh, bh) : row_value<T, MODE>(acc, xh, bh, a.omega, inverse(L[0]));
    if (MODE != kNormB)
      for (int c = lane; c < t.y0; c += kWave) a.Y[L[c].idx] = out;
    if (lane == 0) accum<T, MODE>(ss, mx, out, xh);
    return;
  }
  for (int step = 0; step < 2; ++step) {
    const int n = step == 0 ? t.y0 : t.z;
    if (n == 0) break;
    const bool live = lane < n;
    const EdgeCopy k = L[live ? lane : 0];
    const T inv = inverse(k);
    T p, xo, bo, acc = T(0);
    load(k, live, lane == k.head, p, xo, bo);
    if (kX) {
      const int nc = live ? k.copies : 0;
      for (int i = 0; __builtin_amdgcn_ballot_w64(i < nc); ++i) {
        const T v = __shfl(p, (k.head + i) & (kWave - 1), kWave);
        acc += i < nc ? v : T(0);
      }
    }
    const T xh = __shfl(xo, k.head, kWave), bh = __shfl(bo, k.head, kWave);
    const T out = fixed(k) ? dirichlet_row<T, MODE>(xo, bo) : row_value<T, MODE>(acc, xh, bh, a.omega, inv);
    if (live) {
      if (MODE != kNormB) a.Y[k.idx] = out;
      if (lane == k.head) accum<T, MODE>(ss, mx, out, xo);
    }
    L += t.y0;
  }
}

// y = the sum over its copies of partial(copy) at the 2D shared DoFs of tile t,
// laid out as for edge_rows.
template <typename T, class Partial>
__device__ __forceinline__ void shared_rows(const EdgeCopy* edges, const Tile& t, T* Y, Partial partial) {
  const int lane = threadIdx.x & (kWave - 1);
  const EdgeCopy* L = edges + t.x0;
  if (t.macro == kEdgeBigTile) {
    T acc = T(0);
    for (int c0 = 0; c0 < t.y0; c0 += kWave) {
      const int n = min(kWave, t.y0 - c0);
      const T p = lane < n ? partial(L[c0 + lane]) : T(0);
      for (int i = 0; i < n; ++i) acc += __shfl(p, i, kWave);
    }
    for (int c = lane; c < t.y0; c += kWave) Y[L[c].idx] = acc;
    return;
  }
  for (int step = 0; step < 2; ++step) {
    const int n = step == 0 ? t.y0 : t.z;
    if (n == 0) break;
    const bool live = lane < n;
    const EdgeCopy e = L[live ? lane : 0];
    const T p = live ? partial(e) : T(0);
    T acc = T(0);
    const int nc = live ? e.copies : 0;
    for (int i = 0; __builtin_amdgcn_ballot_w64(i < nc); ++i) {
      const T v = __shfl(p, (e.head + i) & (kWave - 1), kWave);
      acc += i < nc ? v : T(0);
    }
    if (live) Y[e.idx] = acc;
    L += t.y0;
  }
}

}  // namespace mf

// Variable-coefficient P1 apply (gfx950): y = A(k) x with A(k) the
// stiffness matrix of -div(k grad u), k the P1 interpolant of nodal values
// k_i (a vector in storage layout).  On a P1 element grad u . grad v is
// constant, so each element matrix is exactly mean_T(k) times the
// constant-coefficient one; the rows are formed on the fly from the macro's
// two element matrices and the coefficient, which the paper notes as the way
// to keep varying weights matrix-free at the price of extra arithmetic
// (comparison of matrix-free and sparse storage).  Traffic: k and x read,
// y written (24 B/DoF in FP64).
//
// Walk: as the constant-coefficient 2D walk, a wave owns 64 columns (62
// outputs) of a strip of rows and keeps three rows of x and k in registers.
// A point's row sums over its six micro-triangles: U(x,y), U(x-1,y),
// U(x,y-1) (up) and D(x-1,y), D(x-1,y-1), D(x,y-1) (down), where U(a,b) has
// vertices (a,b),(a+1,b),(a,b+1) and D(a,b) has (a+1,b),(a+1,b+1),(a,b+1).
// The triangle coefficients of one band of rows are computed once per lane
// and reused by the two rows that share the band.  Macro-boundary points sum
// only the triangles inside the macro (a partial row, completed for shared
// DoFs by the exchange kernel); Dirichlet points copy x.

#include <hip/hip_runtime.h>

#include <string>

#include "launch.hpp"
#include "rows.hpp"
#include "walk3d.hpp"
#include "wave.hpp"

namespace mf {

namespace {

using wave::dn1;
using wave::up1;

template <typename T>
struct VcTile {
  static constexpr int H = kTileH2, U = 4;
};
template <>
struct VcTile<float> {
  static constexpr int H = kTileH2F, U = 8;
};

// Column xc (>= 0) of row r of a triangle of side N stored at base, with the
// row clamped to [0, min(last, N)] and the column into the row.
template <typename T>
__device__ __forceinline__ T ld_row(const T* __restrict__ base, int N, int r, int last, int xc) {
  const int rr = min(max(r, 0), min(last, N));
  return base[row_start(N, rr) + min(xc, N - rr)];
}

// Coefficients of the up and down triangles with anchor (x, b), from k rows
// b and b+1 of this lane (kb, kb1) and of lane + 1.
template <typename T>
__device__ __forceinline__ void band_coef(T kb, T kb1, T third, T& ku, T& kd) {
  const T kbr = dn1(kb), kb1r = dn1(kb1);
  ku = (kb + kbr + kb1) * third;
  kd = (kbr + kb1r + kb1) * third;
}

template <typename T, bool INNER>
__device__ __forceinline__ void vc_tile(int x0, int y0, const MacroDev& M, const T* __restrict__ K,
                                        const T* __restrict__ X, T* __restrict__ Y) {
  constexpr int kH = VcTile<T>::H, kU = VcTile<T>::U;
  const int lane = threadIdx.x & (kWave - 1);
  const int N = M.N;
  const int x = x0 - 1 + lane;
  const int xc = max(x, 0);
  const int y1 = min(y0 + kH, N - x0 + 1);  // output rows y0 .. y1-1
  K += M.base;
  X += M.base;
  Y += M.base;
  // element matrices: up (type 0) and down (type 1), local rows 0..2
  T ku[3][3], kd[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      ku[i][j] = (T)M.K[0][i * 4 + j];
      kd[i][j] = (T)M.K[1][i * 4 + j];
    }
  const T third = T(1) / T(3);

  // x and k of rows y-1 (m), y (0), y+1 (p); triangle coefficients of bands
  // y-1 (between rows y-1 and y) and y
  T xm = ld_row(X, N, y0 - 1, y1, xc), x0v = ld_row(X, N, y0, y1, xc);
  T km = ld_row(K, N, y0 - 1, y1, xc), k0 = ld_row(K, N, y0, y1, xc);
  T kum, kdm;
  band_coef(km, k0, third, kum, kdm);
  T qx[kU], qk[kU];
#pragma unroll
  for (int j = 0; j < kU; ++j) {
    qx[j] = ld_row(X, N, y0 + 1 + j, y1, xc);
    qk[j] = ld_row(K, N, y0 + 1 + j, y1, xc);
  }
  const int nrows = y1 - y0;
#pragma unroll
  for (int j = 0; j < kH; ++j) {
    const int yy = y0 + j;
    const T xp = qx[j % kU], kp = qk[j % kU];
    qx[j % kU] = ld_row(X, N, y0 + 2 + j + kU - 1, y1, xc);
    qk[j % kU] = ld_row(K, N, y0 + 2 + j + kU - 1, y1, xc);
    if (j >= nrows) continue;
    T kup, kdp;  // band y
    band_coef(k0, kp, third, kup, kdp);
    const T xE = dn1(x0v), xW = up1(x0v), xNW = up1(xp), xSE = dn1(xm);
    const T t1 = ku[0][0] * x0v + ku[0][1] * xE + ku[0][2] * xp;
    const T t2 = ku[1][0] * xW + ku[1][1] * x0v + ku[1][2] * xNW;
    const T t3 = ku[2][0] * xm + ku[2][1] * xSE + ku[2][2] * x0v;
    const T t4 = kd[0][0] * x0v + kd[0][1] * xp + kd[0][2] * xNW;
    const T t5 = kd[1][0] * xm + kd[1][1] * x0v + kd[1][2] * xW;
    const T t6 = kd[2][0] * xSE + kd[2][1] * xE + kd[2][2] * x0v;
    const T c1 = kup, c2 = up1(kup), c3 = kum, c4 = up1(kdp), c5 = up1(kdm), c6 = kdm;
    T acc;
    const bool inside = lane >= 1 && lane <= kTileW && x + yy <= N;
    if (INNER) {
      acc = c1 * t1;
      acc = fma(c2, t2, acc);
      acc = fma(c3, t3, acc);
      acc = fma(c4, t4, acc);
      acc = fma(c5, t5, acc);
      acc = fma(c6, t6, acc);
      if (inside) Y[row_start(N, yy) + xc] = acc;
    } else {
      // triangles inside the macro (the point itself is inside)
      const bool in1 = x + yy <= N - 1, in2 = x >= 1, in3 = yy >= 1;
      const bool in4 = x >= 1 && x + yy <= N - 1, in5 = x >= 1 && yy >= 1, in6 = yy >= 1 && x + yy <= N - 1;
      acc = in1 ? c1 * t1 : T(0);
      acc = in2 ? fma(c2, t2, acc) : acc;
      acc = in3 ? fma(c3, t3, acc) : acc;
      acc = in4 ? fma(c4, t4, acc) : acc;
      acc = in5 ? fma(c5, t5, acc) : acc;
      acc = in6 ? fma(c6, t6, acc) : acc;
      if (inside) {
        const bool dir = (M.dir_mask >> support_mask(2, N, x, yy, 0)) & 1;
        Y[row_start(N, yy) + xc] = dir ? x0v : acc;
      }
    }
    xm = x0v;
    x0v = xp;
    k0 = kp;
    kum = kup;
    kdm = kdp;
  }
}

template <typename T>
__global__ __launch_bounds__(kWG) void varcoef_kernel(const Tile* __restrict__ tiles, int nwg, const MacroDev* md,
                                                      const T* __restrict__ K, const T* __restrict__ X,
                                                      T* __restrict__ Y) {
  const int g = wave::xcd_wg_runs(nwg, wave::kRuns2);
  if (g < 0) return;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Tile t = tiles[g * kWavesPerWG + wv];
  if (t.macro < 0) return;
  const MacroDev& M = md[t.macro];
  if (t.x0 >= 1 && t.y0 >= 1 && t.x0 + t.y0 + kTileW + VcTile<T>::H <= M.N)
    vc_tile<T, true>(t.x0, t.y0, M, K, X, Y);
  else
    vc_tile<T, false>(t.x0, t.y0, M, K, X, Y);
}

template <typename T>
int run_varcoef(const Level& L, const void* k, const void* x, void* y, hipStream_t s) {
  const bool f32 = sizeof(T) == 4 && !L.tiles_f32.empty();
  const Tile* tiles = (f32 ? L.dev.tiles_f32 : L.dev.tiles) + L.ewgs * kWavesPerWG;
  const int nwg = (int)((f32 ? L.tiles_f32.size() : L.tiles.size()) / kWavesPerWG) - L.ewgs;
  // five workgroups per CU on large launches of long rows (level 14: FP64 578.7 -> 560 us, FP32 301.7 -> 283; level 13
  // 151 -> 149, 79.4 -> 78)
  if (nwg > 0)
    hipLaunchKernelGGL(varcoef_kernel<T>, dim3(wave::xcd_grid_runs(nwg, wave::kRuns2)), dim3(kWG),
                       L.N >= wave::kCapN ? wave::lds_cap(nwg, wave::kRuns2.from, 5, 0) : 0, s, tiles, nwg, L.dev.md,
                       (const T*)k, (const T*)x, (T*)y);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(MF_EDEVICE, hipGetErrorString(e));
  return launch_exchange_apply(L, dtype_of<T>(), y, s);
}

// ---------------------------------------------------------------- 3D
template <typename T>
struct VarcoefArgs {
  const Tile* tiles;
  const Tile* btiles;  // the boundary tiles alone
  const MacroDev* md;
  const FaceDev* faces;
  const EdgeCopy* edges;
  const T* K;
  const T* X;
  T* Y;
};

// Tetrahedral macros: columns as in the constant-coefficient walk (walk3d.hpp),
// and one launch for the macro faces, edges and vertices.
//
// Interior points.  The micro-tets come six to a lattice cell (x, y, z) ..
// (x + 1, y + 1, z + 1), types t0 .. t5, and an element matrix has zero row
// sums, so a row is sum_j w_ij (x_j - x_i) over its 14 lattice edges, w_ij
// summing (coefficient sum of the tet) x (entry ij of its matrix) over the
// tets around the edge: 36 products per cell for the seven edges per point,
// each then used by both of its ends, instead of 24 element rows per point.
// The reflection of a cell through its centre maps t0, t1, t2 to t5, t3, t4,
// so 18 entries serve all six.
//
// A lane walks its column layer by layer (the cells between two slices).  A
// layer completes the weights of the edges inside its lower slice (begun by
// the layer below), forms those of the edges across it, and adds every edge's
// flux to its two ends: the lower slice's rows are then complete, the upper
// slice's begun.  Ends and cells in the lane to the left are reached by
// shifting sums.  The 1/4 of the coefficient means is applied once to the row
// (a power of two: exact).
//
// Bound: vector issue and memory about equally.  Cube, against a lane per
// point that gathers 30 values and forms 24 element rows: N = 256 FP64 301 -> 138
// us, FP32 143 -> 75 (24 and 12 B/DoF: 3.0 and 2.7 TB/s), N = 128 46 -> 30 and 27 ->
// 20 (with the boundary in the same launch 126 and 62, 21.4 and 14.1).  More than two
// workgroups per CU spill with bands of two rows in FP64.
template <typename T, int R>
__device__ __forceinline__ void vc_walk3(const Tile& t, const MacroDev& M, const T* __restrict__ K,
                                         const T* __restrict__ X, T* __restrict__ Y) {
  constexpr unsigned E = sizeof(T);
  constexpr int NS = 3;  // slices in registers: a layer's two, and the next
  const int N = uniform(M.N), z0 = t.z & 0xffff, nz = t.z >> 16, A = N - z0;
  const T* P0 = Prec<T>::K(M, 0);
  const T* P1 = Prec<T>::K(M, 1);
  const T* P2 = Prec<T>::K(M, 2);
  const T a01 = uniform(P0[1]), a02 = uniform(P0[2]), a03 = uniform(P0[3]), a12 = uniform(P0[6]), a13 = uniform(P0[7]), a23 = uniform(P0[11]);
  const T b01 = uniform(P1[1]), b02 = uniform(P1[2]), b03 = uniform(P1[3]), b12 = uniform(P1[6]), b13 = uniform(P1[7]), b23 = uniform(P1[11]);
  const T c01 = uniform(P2[1]), c02 = uniform(P2[2]), c03 = uniform(P2[3]), c12 = uniform(P2[6]), c13 = uniform(P2[7]), c23 = uniform(P2[11]);
  const WalkLane wl = walk_lane<R>(t, M);
  const int64_t sb = uniform(M.base) + slice_base(N, z0 - 1);
  const int64_t rest = tet_count_small(N + 1) - slice_base(N, z0 - 1);
  const buf::Rsrc bk = buf::make(K + sb, rest), bx = buf::make(X + sb, rest), by = buf::make(Y + sb, rest);
  Cursor<T> in(A, wl.col), out(A, wl.col);
  out.next();
  T k[NS][R + 2], x[NS][R + 2];  // rows y0 .. y0 + R + 1
  auto load = [&](T* kv, T* xv) {
    unsigned r = in.off;
#pragma unroll
    for (int j = 0; j < R + 2; ++j) {
      kv[j] = buf::ld<T>(bk, r);
      xv[j] = buf::ld<T>(bx, r);
      r += in.row - (unsigned)j * E;
    }
    in.next();
  };
#pragma unroll
  for (int i = 0; i < NS; ++i) load(k[i], x[i]);
  T kr[NS][R + 2], xr[NS][R + 2];  // the same at x + 1
#pragma unroll
  for (int j = 0; j < R + 2; ++j) {
    kr[0][j] = dn1(k[0][j]);
    xr[0][j] = dn1(x[0][j]);
  }
  // begun by the layer below: weights of the lower slice's edges along x, y and x - y, and its rows
  T w1[R + 1], w2[R + 1], w12[R + 1], ys[R + 1];
#pragma unroll
  for (int j = 0; j <= R; ++j) w1[j] = w2[j] = w12[j] = ys[j] = T(0);
  for (int i0 = 0; i0 <= nz; i0 += NS) {
#pragma unroll
    for (int ii = 0; ii < NS; ++ii) {
      const int i = i0 + ii;  // layer between slices z0 - 1 + i and z0 + i
      if (i > nz) break;
      const T *k0 = k[ii], *q0 = kr[ii], *x0 = x[ii], *v0 = xr[ii];
      const T *k1 = k[(ii + 1) % NS], *x1 = x[(ii + 1) % NS];
      T *q1 = kr[(ii + 1) % NS], *v1 = xr[(ii + 1) % NS];
#pragma unroll
      for (int j = 0; j < R + 2; ++j) {
        q1[j] = dn1(k1[j]);
        v1[j] = dn1(x1[j]);
      }
      T lo[R + 2], up[R + 2];  // the layer's share of the lower and of the upper rows
#pragma unroll
      for (int j = 0; j < R + 2; ++j) lo[j] = up[j] = T(0);
      // of the cells one row below: shares of the edges along x (lower and upper slice), z, x - z, and the left lane's z
      T pB = T(0), pD = T(0), pK = T(0), pP = T(0), pL = T(0);
#pragma unroll
      for (int j = 0; j <= R; ++j) {
        // coefficient sums of the cell's tets
        const T body = k0[j + 1] + q1[j], s100_001 = q0[j] + k1[j], s110_011 = q0[j + 1] + k1[j + 1];
        const T t0 = (k0[j] + k0[j + 1]) + s100_001;
        const T t1 = body + (q0[j] + q0[j + 1]);
        const T t2 = body + s110_011;
        const T t3 = body + (k1[j + 1] + k1[j]);
        const T t4 = body + s100_001;
        const T t5 = (q1[j] + q1[j + 1]) + s110_011;
        const bool row = j >= 1;  // (row 0 only feeds row 1)
        // edges of the lower slice, complete with this layer
        const T W2 = w2[j] + (a02 * t0 + up1(b23 * t1));
        const T W12 = w12[j] + fma(c13, t4, fma(b02, t1, a12 * t0));
        // edges across the layer
        const T W23 = fma(c12, t4, fma(b13, t3, a23 * t0)) + up1(fma(a23, t5, fma(c12, t2, b13 * t1)));
        const T Wb = fma(c01, t2 + t4, b01 * (t1 + t3));
        const T d2 = x0[j + 1] - x0[j], d12 = v0[j] - x0[j + 1], d23 = x0[j + 1] - x1[j], db = v1[j] - x0[j + 1];
        T left = T(0);
        if (row) {
          const T W1 = w1[j] + fma(a01, t0, pB);
          const T W3 = (fma(a03, t0, pK)) + up1(fma(c03, t4, fma(b12, t1, pL)));
          const T W13 = fma(c23, t4, fma(a13, t0, pP));
          const T d1 = v0[j] - x0[j], d3 = x1[j] - x0[j], d13 = v0[j] - x1[j];
          lo[j] = fma(W1, d1, lo[j]);
          lo[j] = fma(W2, d2, lo[j]);
          lo[j] = fma(W3, d3, lo[j]);
          left = fma(W13, d13, fma(W12, d12, W1 * d1));
          lo[j] -= up1(left);
          up[j] = fma(W13, d13, up[j]);
          up[j] = fma(-W3, d3, up[j]);
          up[j] = fma(W23, d23, up[j]);
          up[j] -= up1(Wb * db);
        }
        lo[j + 1] = fma(-W2, d2, lo[j + 1]);
        lo[j + 1] = fma(W12, d12, lo[j + 1]);
        lo[j + 1] = fma(-W23, d23, lo[j + 1]);
        lo[j + 1] = fma(Wb, db, lo[j + 1]);
        // edges of the upper slice, begun
        if (row) w1[j] = fma(c02, t4, fma(b03, t3, pD));
        w2[j] = fma(b23, t3, up1(a02 * t5));
        w12[j] = fma(a12, t5, fma(b02, t3, c13 * t2));
        pB = fma(c02, t2, b03 * t1);
        pD = a01 * t5;
        pK = fma(b12, t3, c03 * t2);
        pP = fma(a13, t5, c23 * t2);
        pL = a03 * t5;
      }
      if (i > 0) {
        unsigned r = out.off;
        const int kk = i - 1;
#pragma unroll
        for (int j = 1; j <= R; ++j) {
          r += out.row - (unsigned)(j - 1) * E;
          const T v = wl.copies(j + kk) ? x0[j] : (ys[j] + lo[j]) * T(0.25);
          buf::st<T>(by, wl.writes(j + kk) ? r : buf::kDrop, v);
        }
        out.next();
      }
#pragma unroll
      for (int j = 1; j <= R; ++j) ys[j] = up[j];
      if (i + NS <= nz + 1) load(k[ii], x[ii]);
    }
  }
}

// Macro-boundary points: one lane per point and copy, 24 element rows at most,
// each the coefficient sum of its tet times its row of the element matrix.
// Every vertex of a tet around a point is the point or one of its 15 stencil
// neighbours.  Bound: the gathers (rows of a face lie a slice or a row apart, and
// the copies of edges and vertices have a macro per lane).  A workgroup per tile,
// with a face's two copies in two waves.  Against all 96 entries of
// the six matrices (256 registers in FP64): cube at level 7 FP64 27.7 -> 24.7 us, level
// 8 137 -> 130; 3,072 tets at level 3 FP64 109 -> 43, FP32 35.8 -> 28.1, 384 at level 5
// FP64 87 -> 65.

// Index into the 15 stencil offsets of lattice offset d (-1 if none).
__host__ __device__ constexpr int stencil_slot(int dx, int dy, int dz) {
  constexpr StencilTable ST = stencil_table(3);
  for (int o = 0; o < ST.n; ++o)
    if (ST.off[o][0] == dx && ST.off[o][1] == dy && ST.off[o][2] == dz) return o;
  return -1;
}

// Stencil slot of vertex u of a type-t tet whose vertex v is the point.
__host__ __device__ constexpr int tet_slot(int t, int v, int u) {
  constexpr ElemTable E = elem_table(3);
  return stencil_slot(E.off[t][u][0] - E.off[t][v][0], E.off[t][u][1] - E.off[t][v][1],
                      E.off[t][u][2] - E.off[t][v][2]);
}

__host__ __device__ constexpr bool tet_slots_valid() {
  for (int t = 0; t < 6; ++t)
    for (int v = 0; v < 4; ++v)
      for (int u = 0; u < 4; ++u)
        if (tet_slot(t, v, u) < 0) return false;
  return true;
}
static_assert(tet_slots_valid(), "every edge of a micro-tet is a stencil offset");

// Whether that tet lies in the macro when the point is an inner point of face f.
__host__ __device__ constexpr bool tet_on_side(int f, int t, int v) {
  for (int u = 0; u < 4; ++u)
    if (!on_side(f, tet_slot(t, v, u))) return false;
  return true;
}

// The element matrices' entries by type, vertex and vertex: a matrix is symmetric,
// and type t's is that of type 0, 1 or 2 whose tet t is, or is the reflection of
// through the cell's centre, so 30 entries serve all six (like[t][v][u] among
// them).
struct LikeTable {
  int8_t like[6][4][4];
};
__host__ __device__ constexpr LikeTable like_table() {
  constexpr ElemTable E = elem_table(3);
  LikeTable L{};
  for (int t = 0; t < 6; ++t) {
    int to[4] = {0, 1, 2, 3}, base = t;
    for (int b = 0; b < 3 && t >= 3; ++b) {
      int found = 0;
      for (int v = 0; v < 4; ++v)
        for (int u = 0; u < 4; ++u) {
          bool same = true;
          for (int d = 0; d < 3; ++d) same = same && E.off[b][u][d] == 1 - E.off[t][v][d];
          if (same) to[v] = u, ++found;
        }
      if (found == 4) {
        base = b;
        break;
      }
    }
    for (int v = 0; v < 4; ++v)
      for (int u = 0; u < 4; ++u) {
        const int lo = to[v] < to[u] ? to[v] : to[u], hi = to[v] < to[u] ? to[u] : to[v];
        L.like[t][v][u] = (int8_t)(10 * base + (lo * (7 - lo)) / 2 + hi);
      }
  }
  return L;
}
constexpr bool like_table_valid() {
  constexpr LikeTable L = like_table();
  for (int t = 0; t < 6; ++t)
    for (int v = 0; v < 4; ++v)
      for (int u = 0; u < 4; ++u)
        if (L.like[t][v][u] < 0 || L.like[t][v][u] >= 30 || L.like[t][v][u] != L.like[t][u][v]) return false;
  return true;
}
static_assert(like_table_valid(), "30 entries serve all six types");

// Four times the row of a point from the coefficients and values of its
// stencil neighbours; in(t, v): its type-t tet with the point as vertex v is
// in the macro; UNIFORM: all lanes have the same macro.  (The walk's differences
// against the point would need 18 entries, FP64 3,072 tets at level 3 37 us, but make
// FP32 rows up to 3 % less exact.)
template <bool UNIFORM, typename T, class In>
__device__ __forceinline__ T vc3_row(const MacroDev& M, const T* kv, const T* xv, In in) {
  constexpr ElemTable E = elem_table(3);
  constexpr LikeTable L = like_table();
  T e[30];
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int u = v; u < 4; ++u) {
        const T& k = Prec<T>::K(M, t)[4 * v + u];
        e[L.like[t][v][u]] = UNIFORM ? uniform(k) : k;
      }
  __builtin_amdgcn_sched_barrier(0);  // every load before the sums
  T acc = T(0);
#pragma unroll
  for (int t = 0; t < E.ntypes; ++t) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int s0 = tet_slot(t, v, 0), s1 = tet_slot(t, v, 1), s2 = tet_slot(t, v, 2), s3 = tet_slot(t, v, 3);
      const T ks = kv[s0] + kv[s1] + kv[s2] + kv[s3];
      T r = e[L.like[t][v][0]] * xv[s0];
      r = fma(e[L.like[t][v][1]], xv[s1], r);
      r = fma(e[L.like[t][v][2]], xv[s2], r);
      r = fma(e[L.like[t][v][3]], xv[s3], r);
      acc = in(t, v) ? fma(ks, r, acc) : acc;
    }
  }
  return acc;
}

template <typename T, int F>
__device__ __forceinline__ T vc3_face(const MacroDev& M, const T* K, const T* X, int N, int y, int z) {
  int off[15];
  nbr_offsets3(N, y, z, off);
  T kv[15], xv[15];
#pragma unroll
  for (int o = 0; o < 15; ++o) {
    kv[o] = on_side(F, o) ? K[off[o]] : T(0);
    xv[o] = on_side(F, o) ? X[off[o]] : T(0);
  }
  return vc3_row<true>(M, kv, xv, [](int t, int v) { return tet_on_side(F, t, v); });
}

// One tile of the macro boundary per workgroup.  Faces of two macros: waves 2 c
// and 2 c + 1 take the two copies of the tile's c-th 64 points and add their
// rows through LDS, so no wave waits for one copy's gathers before the
// other's.
template <typename T>
__device__ __forceinline__ void vc3_faces(const VarcoefArgs<T>& a, const Tile& t, int wv, T* part) {
  const FaceDev& F = a.faces[t.z];
  const int lane = threadIdx.x & (kWave - 1);
  if (F.dirichlet) {
    for (int i = threadIdx.x; i < t.y0; i += kWG) {
      int ia, ib, x, y, z;
      slice_xy3(F.N - 3, t.x0 + i, ia, ib);
      const int64_t p = face_index(a.md, F.cp[0], F.N, ia + 1, ib + 1, x, y, z);
      a.Y[p] = a.X[p];
    }
    return;
  }
  const bool two = F.copies == 2;
  const int c = two ? wv & 1 : 0, step = two ? kWG / 2 : kWG;
  const FaceCopy& C = F.cp[c];
  const MacroDev& M = a.md[C.macro];
  for (int i0 = 0; i0 < t.y0; i0 += step) {
    const int i = i0 + (two ? wv >> 1 : wv) * kWave + lane;
    int ia, ib, x, y, z;
    slice_xy3(F.N - 3, t.x0 + min(i, t.y0 - 1), ia, ib);
    const int64_t p = face_index(a.md, C, F.N, ia + 1, ib + 1, x, y, z);
    T acc;
    switch (C.face) {
      case 0: acc = vc3_face<T, 0>(M, a.K + p, a.X + p, F.N, y, z); break;
      case 1: acc = vc3_face<T, 1>(M, a.K + p, a.X + p, F.N, y, z); break;
      case 2: acc = vc3_face<T, 2>(M, a.K + p, a.X + p, F.N, y, z); break;
      default: acc = vc3_face<T, 3>(M, a.K + p, a.X + p, F.N, y, z); break;
    }
    if (two) {
      part[threadIdx.x] = acc;
      __syncthreads();
      acc = part[(wv & ~1) * kWave + lane] + part[(wv | 1) * kWave + lane];
      __syncthreads();
    }
    if (i < t.y0) a.Y[p] = acc * T(0.25);
  }
}

template <typename T>
__device__ __forceinline__ T vc3_copy(const VarcoefArgs<T>& a, const EdgeCopy& e) {
  constexpr StencilTable ST = stencil_table(3);
  constexpr ElemTable E = elem_table(3);
  const MacroDev& M = a.md[e.macro];
  const int N = M.N;
  int off[15];
  nbr_offsets3(N, e.y, e.z, off);
  T kv[15], xv[15];
#pragma unroll
  for (int o = 0; o < 15; ++o) {
    const int nx = e.x + ST.off[o][0], ny = e.y + ST.off[o][1], nz = e.z + ST.off[o][2];
    const bool in = nx >= 0 && ny >= 0 && nz >= 0 && nx + ny + nz <= N;
    const int64_t i = in ? e.idx + off[o] : e.idx;  // (no tet uses the neighbours outside)
    kv[o] = a.K[i];
    xv[o] = a.X[i];
  }
  return vc3_row<false>(M, kv, xv, [&](int t, int v) {
    const int ax = e.x - E.off[t][v][0], ay = e.y - E.off[t][v][1], az = e.z - E.off[t][v][2];
    return ax >= 0 && ay >= 0 && az >= 0 && ax + ay + az <= N - E.slack[t];
  });
}

template <typename T>
__device__ __forceinline__ void vc3_edges(const VarcoefArgs<T>& a, const Tile& t) {
  const int lane = threadIdx.x & (kWave - 1);
  const EdgeCopy* L = a.edges + t.x0;
  if (t.macro == kEdgeBigTile) {
    T acc = T(0);
    if (!L[0].dirichlet)
      for (int c0 = 0; c0 < t.y0; c0 += kWave) {
        const int n = min(kWave, t.y0 - c0);
        const T p = lane < n ? vc3_copy<T>(a, L[c0 + lane]) : T(0);
        for (int i = 0; i < n; ++i) acc += __shfl(p, i, kWave);
      }
    for (int c = lane; c < t.y0; c += kWave) a.Y[L[c].idx] = L[0].dirichlet ? a.X[L[c].idx] : acc * T(0.25);
    return;
  }
  const bool live = lane < t.y0;
  const EdgeCopy e = L[live ? lane : 0];
  T p = T(0), acc = T(0);
  if (live && !e.dirichlet) p = vc3_copy<T>(a, e);
  const int n = live ? e.copies : 0;
  for (int i = 0; __builtin_amdgcn_ballot_w64(i < n); ++i) {
    const T v = __shfl(p, (e.head + i) & (kWave - 1), kWave);
    acc += i < n ? v : T(0);
  }
  if (live) a.Y[e.idx] = e.dirichlet ? a.X[e.idx] : acc * T(0.25);
}

// One launch: the boundary's workgroups first (its gathers wait while the walk
// streams), then the walk's.  Against a launch each: a tet at levels 6 and 7 FP64 9.4 and
// 9.9 -> 5.7 and 6.2 us, FP32 8.8 and 9.1 -> 5.2 and 5.4; the cube at level 7 24.8 ->
// 21.4, at level 8 130 -> 126 and 65 -> 62.  In FP64 the boundary needs more registers
// than bands of one row; held to 168 (none spill) both keep three workgroups per CU: 384
// tets at level 5 54.4 us (64 as two launches, 67 at 170 registers and two workgroups),
// 3,072 at level 3 33.2 (43).
template <typename T, int R>
__global__ __launch_bounds__(kWG, R == 1 ? 3 : 2) void varcoef3d_kernel(const VarcoefArgs<T> a, int nb, int nwg) {
  __shared__ T part[kWG];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), head = wave::xcd_grid(nb);
  if ((int)blockIdx.x < head) {
    if ((int)blockIdx.x >= nb) return;
    const Tile t = load_seg(a.btiles, blockIdx.x);
    if (t.macro == kFaceTile) vc3_faces<T>(a, t, wv, part);
    else if (t.macro != -1 && wv == 0) vc3_edges<T>(a, t);
    return;
  }
  const int g = wave::xcd_wg_at(blockIdx.x - head, nwg, wave::kRuns3);
  if (g < 0) return;
  const Tile t = load_seg(a.tiles, g * kWavesPerWG + wv);
  if (t.macro >= 0) vc_walk3<T, R>(t, a.md[t.macro], a.K, a.X, a.Y);
}

// Bands of R rows: those of shape3_varcoef (FP64 up to 2, FP32 up to 3).
template <typename T, int R = sizeof(T) == 8 ? 2 : 3>
int run_vc3(int rows, const VarcoefArgs<T>& a, int nb, int nwg, hipStream_t s) {
  if (rows == R) {
    const dim3 grid(wave::xcd_grid(nb) + wave::xcd_grid_runs(nwg, wave::kRuns3));
    hipLaunchKernelGGL((varcoef3d_kernel<T, R>), grid, dim3(kWG), 0, s, a, nb, nwg);
    return MF_OK;
  }
  if constexpr (R > 1) return run_vc3<T, R - 1>(rows, a, nb, nwg, s);
  else return set_error(MF_EINVAL, "internal: no variable-coefficient walk over bands of " + std::to_string(rows) + " rows");
}

template <typename T>
int run_varcoef3d(const Level& L, const void* k, const void* x, void* y, hipStream_t s) {
  constexpr int i = sizeof(T) == 8 ? 0 : 1;
  const int nb = (int)L.btiles.size(), nwg = (int)(L.vtiles[i].size() / kWavesPerWG);
  const VarcoefArgs<T> a{L.dev.vtiles[i], L.dev.btiles, L.dev.md, L.dev.faces, L.dev.edges,
                         (const T*)k,      (const T*)x,   (T*)y};
  if (nb + nwg > 0)
    if (const int rc = run_vc3<T>(shape3_varcoef(L.N, i == 1).R, a, nb, nwg, s)) return rc;
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? MF_OK : set_error(MF_EDEVICE, hipGetErrorString(e));
}

}  // namespace

int launch_varcoef_apply(const mf_mesh* m, const Level& L, int dtype, const void* k, const void* x, void* y,
                         hipStream_t s) {
  if (m->dim == 3)
    return dtype == MF_F64 ? run_varcoef3d<double>(L, k, x, y, s) : run_varcoef3d<float>(L, k, x, y, s);
  return dtype == MF_F64 ? run_varcoef<double>(L, k, x, y, s) : run_varcoef<float>(L, k, x, y, s);
}

}  // namespace mf

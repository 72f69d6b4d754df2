// Constant-stencil kernels for CDNA4 (gfx950): the 2D operator's rows for every
// point of every macro (apply, weighted Jacobi, residual + norm partials),
// the sums over shared DoFs of the variable-coefficient walk, and the
// deterministic norm reduction.
//
// The paper's vertex-to-vertex kernel (Performance Modeling section) walks
// one triangle row by row, x fastest, reading seven neighbours with constant
// weights; on a CPU its speed depends on whether three source rows plus the
// destination row fit in a cache level (the layer condition).  Here the same
// reuse is kept in registers: a 64-lane wavefront owns 64 consecutive
// columns and walks rows upward, holding the rows the stencil needs and taking
// the x+-1 neighbours from adjacent lanes through DPP shifts, so each source
// value is read from memory once per tile; future rows are loaded ahead to
// keep enough bytes in flight for HBM3E (the 3D walk: walk3d.hpp and
// stencil3d_kernels.hip).  No matrix cores: the path is
// HBM-bound.
//
// Macro-boundary DoFs are handled in the same walk (the paper leaves them to
// interface primitives, Performance Modeling, experiment description): a
// point on a face, edge or vertex of its macro uses the partial stencil of
// its support mask — only the micro-elements on its side.  DoFs shared by
// several macros are left to tiles of their own in the same launch (edges.hpp),
// which sum the copies' partial rows in fixed macro order and write the result
// to every copy.

#include <hip/hip_runtime.h>

#include <string>

#include "edges.hpp"
#include "launch.hpp"
#include "rows.hpp"
#include "wave.hpp"

namespace mf {

namespace {

using wave::dn1;
using wave::up1;

// Rows loaded ahead by a tile of H rows.
constexpr int ring2(int H) { return H < 8 ? H : 8; }

static_assert(kTileH2 % ring2(kTileH2) == 0 && kTileH2F % ring2(kTileH2F) == 0, "ring depth must divide the tile height");

// A constant of the macro, the same for every lane.  Beside the shared DoFs' path
// the compiler no longer reads it as a scalar by itself.  Held per lane, FP64 kernels
// need 14 to 16 registers more and lose a wave per SIMD (one triangle at level 12:
// residual 36.2 us, 33.5 as scalars; norm of a residual 55.0 and 49.5).  In FP32 they
// reach eight waves either way, and the walk waits longer for the scalars (Jacobi at
// level 11, two sweeps: 20.7 us and 21.6).
template <typename T, class V>
__device__ __forceinline__ V macro_const(const V& v) {
  if constexpr (sizeof(T) == 8) return uniform(v);
  else return v;
}

// A single mesh without shared DoFs takes to runs later: one triangle at level 12, FP64
// apply / two Jacobi sweeps / residual 22.5 / 64.3 / 32.4 us against 23.6 / 66.2 / 33.3
// in runs.  With shared DoFs in the launch there is no one line: up to 6,000 workgroups
// five triangles at level 11 would gain 4 %, 20 at level 10 would lose 2 % and 3,200
// at level 6 in FP32 7 to 11 %.
template <class A>
MF_HD wave::XcdRuns runs2(const Launch<A>& l) {
  return wave::XcdRuns{l.nseg > 0 || l.lead > 0 ? wave::kRuns2.from : 2 * wave::kRuns2.from, wave::kRuns2.shift};
}

// Copies the 16 x 16 partial-stencil table of macro M into W with `nthreads`
// threads starting at `first` (a wave or the whole workgroup).
template <typename T>
__device__ __forceinline__ void load_wtab(const MacroDev& M, WTab<T> W, int first, int nthreads) {
  for (int i = (int)threadIdx.x - first; i < 256; i += nthreads)
    if (i >= 0) W[i >> 4][i & 15] = Prec<T>::w(M, i >> 4, i & 15);
}

// Interior finish of one row value (full stencil, interior point).
template <typename T, int MODE>
__device__ __forceinline__ void finish_interior(const MacroDev& M, T acc, T xc, T bv, T omega, T* yp, double& ss,
                                                double& mx) {
  T out;
  if (MODE == kApply || MODE == kApplyDot) out = acc;
  else if (MODE == kJacobi || MODE == kJacobi2) out = fma(omega * macro_const<T>(Prec<T>::invd(M)), bv - acc, xc);
  else if (MODE == kResidual) out = bv - acc;
  else out = bv;
  if (MODE != kNormB) st(yp, out);
  accum<T, MODE>(ss, mx, out, xc);
}

// Support masks of the boundary lanes of rows off the y = 0 edge: the row's
// first point (x = 0), its last (far edge) or both.
struct RowMasks {
  static constexpr int L = full_mask(2) & ~2;   // x = 0
  static constexpr int F = full_mask(2) & ~1;   // far edge
  static constexpr int LF = full_mask(2) & ~3;  // both
};

// Row of one point from its neighbour values v (xc = its x, bv = its b).
// may_edge (a compile-time constant after unrolling) marks the rows that can
// lie on the y = 0 edge: those go through the general per-lane path.  In other
// rows a boundary lane is the row's first point (x = 0, only in tiles starting
// at x0 = 0, tile_left), its last (on the far edge x + y = N), or both.  A row
// without such a lane takes the interior stencil (macro_const), and so
// does a row whose boundary lanes are all Dirichlet (they copy x) or shared
// points (written by the edge tiles).  Any
// other row takes, in every lane, the partial stencil of the lane's own
// support mask from the LDS table (interior lanes read the full stencil there,
// the same weights); the neighbours such a lane lacks (x - 1 for x = 0, the
// offsets of coordinate sum +1 on the far edge) have weight 0 in its table
// row, and their stand-in values are replaced by 0 so that those terms add
// exactly nothing.  The terms are summed in table order in every case, so a
// boundary row is the sum over the neighbours it has, in that order.  Jacobi
// needs bid = 1 / centre weight of the L, F and LF masks.
template <typename T, int MODE>
__device__ __forceinline__ void point_row(const MacroDev& M, const WTab<T> W, const T* wi, bool inside, int N, int x,
                                          int y, const T* v, T xc, T bv, T omega, T* yp, double& ss, double& mx,
                                          bool may_edge, bool tile_left, const T* bid) {
  constexpr StencilTable ST = stencil_table(2);
  constexpr int FM = full_mask(2);
  constexpr int NO = ST.n;
  if (may_edge && y == 0) {
    // the row on the y = 0 edge: every lane is a boundary point
    if (__builtin_amdgcn_ballot_w64(inside)) {
      const int mask = support_mask(2, N, x, y, 0);
      const T acc = partial_sum<T, 2>(W, inside ? mask : FM, N, x, y, 0, v);
      const bool shared = ((M.shared_mask & ~M.dir_mask) >> mask) & 1;
      if (inside && !shared) finish<T, 2, MODE>(M, W, mask, acc, xc, bv, omega, yp, ss, mx);
    }
    return;
  }
  const bool far = inside && x + y == N;
  const bool left = tile_left && inside && x == 0;
  if (!__builtin_amdgcn_ballot_w64(far || left)) {
    T acc = wi[0] * v[0];
#pragma unroll
    for (int o = 1; o < NO; ++o) acc = fma(wi[o], v[o], acc);
    if (inside) finish_interior<T, MODE>(M, acc, xc, bv, omega, yp, ss, mx);
    return;
  }
  const bool bnd = far || left;
  const int bm = FM & ~(far ? 1 : 0) & ~(left ? 2 : 0);
  const bool dir = bnd && ((M.dir_mask >> bm) & 1);
  const bool shared = bnd && !dir && ((M.shared_mask >> bm) & 1);
  T a = T(0);
  if (!__builtin_amdgcn_ballot_w64(bnd && !dir && !shared)) {
    // the row's boundary lanes are all Dirichlet (they copy x) or shared (not
    // written): the others take the interior stencil
    a = wi[0] * v[0];
#pragma unroll
    for (int o = 1; o < NO; ++o) a = fma(wi[o], v[o], a);
  } else {
    const T* wr = W[bm];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      T vo = v[o];
      if (ST.off[o][0] + ST.off[o][1] > 0) vo = far ? T(0) : vo;
      if (ST.off[o][0] < 0) vo = left ? T(0) : vo;
      a = o == 0 ? wr[0] * vo : fma(wr[o], vo, a);
    }
  }
  const bool own = !bnd || ((M.own_mask >> bm) & 1);
  T out;
  if (MODE == kApply || MODE == kApplyDot) {
    out = dir ? xc : a;
  } else if (MODE == kJacobi || MODE == kJacobi2) {
    const T id = !bnd ? Prec<T>::invd(M) : far ? (left ? bid[2] : bid[1]) : bid[0];
    out = dir ? (MODE == kJacobi2 ? T(0) : xc) : fma(omega * id, bv - a, xc);
  } else if (MODE == kResidual) {
    out = dir ? bv - xc : bv - a;
  } else {
    out = bv;
  }
  if (inside && !shared) {
    if (MODE != kNormB) st(yp, out);
    if (!dir || own) accum<T, MODE>(ss, mx, out, xc);
  }
}

// ------------------------------------------------------------------ row loads
// Start of row y in a triangle of side S in 32-bit arithmetic (exact for
// every supported level: S <= 32768).
__device__ __forceinline__ int rs32(int S, int y) { return y * (S + 2) - ((y * (y + 1)) >> 1); }

// Value at column xc (>= 0) of row r of a triangle of side S stored at base,
// with the row clamped to [0, last] and the column into the row: a valid
// point for every lane, so loads need no predicate and the unrolled loops
// stay straight-line code (clamped values are never used).  The row address
// is wave-uniform (scalar registers); only the unsigned column offset is per
// lane.
template <typename T>
__device__ __forceinline__ T ldrow(const T* __restrict__ base, int S, int r, int last, int xc) {
  // the row is clamped into [0, S] as well: `last` may name the row past the
  // triangle's apex, and the column offset must stay non-negative
  const int rr = min(max(r, 0), min(last, S));
  const unsigned byte = (unsigned)min(xc, S - rr) * (unsigned)sizeof(T);
  return *(const T*)((const char*)(base + rs32(S, rr)) + byte);
}

// ------------------------------------------------------------------ 2D tile
template <typename T, int MODE, int H>
__device__ __forceinline__ void tile2d(const int x0, const int y0, const MacroDev& M, WTab<T> W,
                                       const T* __restrict__ X, T* __restrict__ Y, const T* __restrict__ B,
                                       T omega, double& ss, double& mx) {
  constexpr int FM = full_mask(2);
  const int lane = threadIdx.x & (kWave - 1);
  const int N = macro_const<T>(M.N);
  const int x = x0 - 1 + lane;
  constexpr int kH = H, kU = ring2(H);
  const int y1 = min(y0 + kH, N - x0 + 1);  // rows y0 .. y1-1 (x0 + y <= N)
  const int64_t base = macro_const<T>(M.base);
  X += base;
  Y += base;
  constexpr bool kZ = MODE == kJacobi2;  // X is b: scaled to the iterate when its row is first used
  constexpr bool kB = MODE != kApply && !kZ;
  if (kB) B += base;
  T wi[7];
#pragma unroll
  for (int o = 0; o < 7; ++o) wi[o] = macro_const<T>(Prec<T>::row(M, FM)[o]);
  T bid[3] = {T(0), T(0), T(0)};
  if (MODE == kJacobi || MODE == kJacobi2) {
    constexpr int c = stencil_table(2).centre;
    bid[0] = T(1) / W[RowMasks::L][c];
    bid[1] = T(1) / W[RowMasks::F][c];
    bid[2] = T(1) / W[RowMasks::LF][c];
  }

  const int xc = max(x, 0);
  T am = ldrow(X, N, y0 - 1, y1, xc);
  T a0 = ldrow(X, N, y0, y1, xc);
  // kJacobi2: omega / diagonal of the column's points inside and on the far
  // edge, and on y = 0 (row y0 of a tile at y0 = 0); raw = b of row y0
  T zi = T(0), zf = T(0), raw = a0;
  if (kZ) {
    const int mx = x <= 0 ? 0 : 2;
    auto c = [&](int mask) { return omega * Prec<T>::zinv(M, mask); };
    zi = c(5 | mx), zf = c(4 | mx);
    am *= x + y0 - 1 == N ? zf : zi;
    a0 *= y0 == 0 ? (x == N ? c(mx) : c(1 | mx)) : (x + y0 == N ? zf : zi);
  }
  T am_r = dn1(am), a0_l = up1(a0), a0_r = dn1(a0);
  T q[kU], qb[kU];
#pragma unroll
  for (int k = 0; k < kU; ++k) {
    q[k] = ldrow(X, N, y0 + 1 + k, y1, xc);                    // x rows y0+1 ..
    if (kB) qb[k] = ldrow(B, N, y0 + k, y1 - 1, xc);  // b rows = output rows
  }
  // The tile's rows are fully unrolled so that the load ring needs no
  // register copies at a loop back-edge (which would wait for every load in
  // flight).  Loads are unconditional; rows past the tile's end only skip
  // the arithmetic (a uniform branch).
  const int nrows = y1 - y0;
#pragma unroll
  for (int k = 0; k < kH; ++k) {
    const int yy = y0 + k;
    const T rp = q[k % kU], ap = kZ ? rp * (x + yy + 1 == N ? zf : zi) : rp;
    const T bv = kZ ? raw : (kB ? qb[k % kU] : T(0));
    raw = rp;
    // (compile-time guards: a ring slot is refilled only if a later row of
    // this tile reads it)
    if (k + kU < kH) q[k % kU] = ldrow(X, N, y0 + 1 + k + kU, y1, xc);
    if (kB && k + kU < kH) qb[k % kU] = ldrow(B, N, y0 + k + kU, y1 - 1, xc);
    if (k >= nrows) continue;
    const T ap_l = up1(ap), ap_r = dn1(ap);
    const T v[7] = {am, am_r, a0_l, a0, a0_r, ap_l, ap};
    const bool inside = lane >= 1 && lane <= kTileW && x + yy <= N;
    point_row<T, MODE>(M, W, wi, inside, N, x, yy, v, a0, bv, omega, Y + rs32(N, yy) + (unsigned)xc, ss, mx, k == 0,
                       x0 == 0, bid);
    am = a0;
    am_r = a0_r;
    a0 = ap;
    a0_l = ap_l;
    a0_r = ap_r;
  }
}

// Interior 2D tile: every row y0-1 .. y0+H exists and holds every column
// x0-1 .. x0+62, and no output point lies on the macro's boundary.  Row
// addresses are then advanced incrementally (row y+1 starts N+1-y entries
// after row y) with no clamping, and every output lane takes the interior
// finish.
// (kJacobi2: nor does any row it reads hold such a point)
template <int H, int MODE>
__device__ __forceinline__ bool tile2d_inner(int x0, int y0, int N) {
  constexpr int in = MODE == kJacobi2 ? 1 : 0;
  return x0 >= 1 + in && y0 >= 1 + in && x0 + y0 + kTileW + H + in <= N;
}

template <typename T, int MODE, int H>
__device__ __forceinline__ void tile2d_fast(const int x0, const int y0, const MacroDev& M, const T* __restrict__ X,
                                            T* __restrict__ Y, const T* __restrict__ B, T omega, double& ss,
                                            double& mx) {
  constexpr int kH = H, kU = ring2(H);
  const int lane = threadIdx.x & (kWave - 1);
  const int N = macro_const<T>(M.N);
  const bool out_lane = (unsigned)(lane - 1) < (unsigned)kTileW;
  const unsigned col = (unsigned)(x0 - 1 + lane) * (unsigned)sizeof(T);
  T wi[7];
#pragma unroll
  for (int o = 0; o < 7; ++o) wi[o] = macro_const<T>(Prec<T>::row(M, full_mask(2))[o]);
  // cursors: byte address of the next row and the byte step to the one after
  const int64_t base = macro_const<T>(M.base);
  const char* px = (const char*)(X + base + rs32(N, y0 - 1));
  int sx = (N + 2 - y0) * (int)sizeof(T);
  char* py = (char*)(Y + base + rs32(N, y0));
  int sy = (N + 1 - y0) * (int)sizeof(T);
  constexpr bool kZ = MODE == kJacobi2, kB = MODE != kApply && !kZ;
  const T zi = kZ ? omega * Prec<T>::zinv(M, full_mask(2)) : T(1);
  const char* pb = kB ? (const char*)(B + base + rs32(N, y0)) : nullptr;
  int sb = sy;
  auto ldx = [&]() -> T {
    const T v = *(const T*)(px + col);
    px += sx;
    sx -= (int)sizeof(T);
    return v;
  };
  auto ldb = [&]() -> T {
    const T v = *(const T*)(pb + col);
    pb += sb;
    sb -= (int)sizeof(T);
    return v;
  };
  T am = ldx();
  T a0 = ldx(), raw = a0;
  if (kZ) am *= zi, a0 *= zi;
  T am_r = dn1(am), a0_l = up1(a0), a0_r = dn1(a0);
  T q[kU], qb[kU];
#pragma unroll
  for (int k = 0; k < kU; ++k) {
    q[k] = ldx();
    if (kB) qb[k] = ldb();
  }
#pragma unroll
  for (int k = 0; k < kH; ++k) {
    const T rp = q[k % kU], ap = kZ ? rp * zi : rp;
    const T bv = kZ ? raw : (kB ? qb[k % kU] : T(0));
    raw = rp;
    if (k + 1 + kU <= kH) q[k % kU] = ldx();
    if (kB && k + kU < kH) qb[k % kU] = ldb();
    const T ap_l = up1(ap), ap_r = dn1(ap);
    const T v[7] = {am, am_r, a0_l, a0, a0_r, ap_l, ap};
    T acc = wi[0] * v[0];
#pragma unroll
    for (int o = 1; o < 7; ++o) acc = fma(wi[o], v[o], acc);
    if (out_lane) finish_interior<T, MODE>(M, acc, a0, bv, omega, (T*)(py + col), ss, mx);
    py += sy;
    sy -= (int)sizeof(T);
    am = a0;
    am_r = a0_r;
    a0 = ap;
    a0_l = ap_l;
    a0_r = ap_r;
  }
}

// Whether a wave tile has output points on its macro's boundary (x = 0, y = 0
// or the far edge x + y = N).
template <int H>
__device__ __forceinline__ bool tile_on_boundary(const Tile& t, int N) {
  return t.x0 == 0 || t.y0 == 0 || t.x0 + t.y0 + (kTileW - 1) + (H - 1) >= N;
}

template <typename T, int MODE, int H>
__global__ __launch_bounds__(kWG) void stencil_kernel(const Launch<StencilArgs<T>> L) {
  const int g = wave::xcd_wg_lead(L.nwg, L.lead, 0, runs2(L));
  if (g < 0) return;
  StencilArgs<T> a;
  const int n = resolve(L, g, a);
  // wave-uniform tile index: every lane reads the same tile and macro constants
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ti = n * kWavesPerWG + wv;
  const Tile t = a.tiles[ti];
  __shared__ T wtab[kWavesPerWG][16][16];
  // The partial-stencil table is only read by tiles that reach the macro's
  // boundary.  The workgroup's four tiles usually share one macro: then one
  // table serves all waves (one load per thread), loaded only if one of the
  // four tiles needs it; otherwise each wave loads its own when it needs it.
  const int m0 = a.tiles[n * kWavesPerWG].macro, m3 = a.tiles[n * kWavesPerWG + kWavesPerWG - 1].macro;
  const bool same = m0 == m3;
  if (same) {
    bool need = false;
    if (m0 >= 0) {
      const int N0 = macro_const<T>(a.md[m0].N);
#pragma unroll
      for (int k = 0; k < kWavesPerWG; ++k) need = need || tile_on_boundary<H>(a.tiles[n * kWavesPerWG + k], N0);
    }
    if (need) {
      load_wtab<T>(a.md[m0], wtab[0], 0, kWG);
      __syncthreads();
    }
  } else if (t.macro >= 0 && tile_on_boundary<H>(t, macro_const<T>(a.md[t.macro].N))) {
    load_wtab<T>(a.md[t.macro], wtab[wv], wv * kWave, kWave);
    __builtin_amdgcn_wave_barrier();
  }
  double ss = 0.0, mx = 0.0;
  if (t.macro >= 0) {
    const MacroDev& M = a.md[t.macro];
    WTab<T> W = wtab[same ? 0 : wv];
    if (tile2d_inner<H, MODE>(t.x0, t.y0, macro_const<T>(M.N))) tile2d_fast<T, MODE, H>(t.x0, t.y0, M, a.X, a.Y, a.B, a.omega, ss, mx);
    else tile2d<T, MODE, H>(t.x0, t.y0, M, W, a.X, a.Y, a.B, a.omega, ss, mx);
  } else if (t.macro != -1) {
    edge_rows<T, 2, MODE>(a, t, ss, mx);
  }
  if (has_partials(MODE) && a.part != nullptr) wg_partial<kWavesPerWG>(ss, mx, a.part, a.np, n);
}

// ------------------------------------------------------------------ exchange

// One DoF shared by several macros and not Dirichlet: its copies hold partial
// rows of the variable-coefficient walk, or the macros' parts of a restriction; sum
// them in fixed macro order and write the row to every copy.  (With tiles of edge
// copies in the walk's own launch, as the other 2D passes have them, that walk was
// slower on large levels: five triangles at level 11 54.0 -> 60.9 us, though seven at
// level 7 took 5.9 instead of 7.8.)
template <typename T>
__global__ __launch_bounds__(kIfaceWG) void exchange_kernel(const GroupArgs<T> a) {
  const int g = blockIdx.x * kIfaceWG + threadIdx.x;
  if (g < a.ngroups) exchange_row(a, g);
}

// y = b at the Dirichlet DoFs (b == NULL: 0).
template <typename T>
__global__ __launch_bounds__(kIfaceWG) void iface_kernel(const Launch<GroupArgs<T>> L) {
  GroupArgs<T> a;
  const int blk = resolve(L, (int)blockIdx.x, a);
  const int g = blk * kIfaceWG + threadIdx.x;
  if (g >= a.ngroups) return;
  const int c0 = a.gptr[g], c1 = a.gptr[g + 1];
  if (!(a.gflag[g] & 1)) return;
  const T v = a.B ? a.B[a.cidx[c0]] : T(0);
  for (int c = c0; c < c1; ++c) a.Y[a.cidx[c]] = v;
}

// result = (sum of part[0, np), max of part[np, 2 np)) in a fixed order; one
// block of kRedT threads per request, four loads in flight per thread.
constexpr int kRedT = 512;
__global__ __launch_bounds__(kRedT) void reduce_kernel(const Launch<ReduceArgs> L) {
  ReduceArgs r;
  resolve(L, (int)blockIdx.x, r);
  __shared__ double s[kRedT], m[kRedT];
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0, b = 0.0;
  int64_t i = threadIdx.x;
  for (; i + 3 * kRedT < r.np; i += 4 * kRedT) {
    a0 += r.part[i];
    a1 += r.part[i + kRedT];
    a2 += r.part[i + 2 * kRedT];
    a3 += r.part[i + 3 * kRedT];
    b = fmax(fmax(b, fmax(r.part[r.np + i], r.part[r.np + i + kRedT])),
             fmax(r.part[r.np + i + 2 * kRedT], r.part[r.np + i + 3 * kRedT]));
  }
  for (; i < r.np; i += kRedT) {
    a0 += r.part[i];
    b = fmax(b, r.part[r.np + i]);
  }
  s[threadIdx.x] = (a0 + a1) + (a2 + a3);
  m[threadIdx.x] = b;
  __syncthreads();
  for (int w = kRedT / 2; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s[threadIdx.x] += s[threadIdx.x + w];
      m[threadIdx.x] = fmax(m[threadIdx.x], m[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double second = r.shift ? r.result[0] : m[0];
    r.result[0] = s[0];
    r.result[1] = second;
    if (r.copy) {
      r.copy[0] = s[0];
      r.copy[1] = second;
    }
  }
}

int check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(MF_EDEVICE, hipGetErrorString(e));
  return MF_OK;
}

// FP32 launches that also read b, on levels whose tiles are mostly interior (N from
// kCapN on; a batch passes 0): five workgroups per CU (one triangle at level 14,
// Jacobi 298.0 -> 290.6 us; the applies and FP64 lose or gain nothing).  Tiles on a
// macro's boundary wait for more than their rows (kCapN).
template <typename T, int MODE>
int stencil_lds(int nwg, int N) {
  constexpr bool pays = sizeof(T) == 4 && MODE != kApply && MODE != kApplyDot;
  constexpr int own = sizeof(T) * kWavesPerWG * 256 + partials_lds(MODE);
  return pays && N >= wave::kCapN ? wave::lds_cap(nwg, wave::kRuns2.from, 5, own) : 0;
}

template <typename T, int MODE>
int run_stencil(int rows, int N, const Launch<StencilArgs<T>>& l, hipStream_t s) {
  if (l.nwg <= 0) return MF_OK;
  const dim3 grid(wave::xcd_grid(l.nwg, l.lead, 0, runs2(l))), wg(kWG);
  const int lds = stencil_lds<T, MODE>(l.nwg, N);
  if (rows == kTileShort[0]) {
    hipLaunchKernelGGL((stencil_kernel<T, MODE, kTileShort[0]>), grid, wg, lds, s, l);
  } else if (rows == kTileShort[1]) {
    hipLaunchKernelGGL((stencil_kernel<T, MODE, kTileShort[1]>), grid, wg, lds, s, l);
  } else if (rows == kTileH2) {
    hipLaunchKernelGGL((stencil_kernel<T, MODE, kTileH2>), grid, wg, lds, s, l);
  } else {
    if constexpr (sizeof(T) == 4) {
      if (rows == kTileH2F) {
        hipLaunchKernelGGL((stencil_kernel<T, MODE, kTileH2F>), grid, wg, lds, s, l);
        return check_launch();
      }
    }
    return set_error(MF_EINVAL, "internal: no 2D walk over tiles of " + std::to_string(rows) + " rows");
  }
  return check_launch();
}

template <typename T>
int run_stencil(int mode, int rows, int N, const Launch<StencilArgs<T>>& l, hipStream_t s) {
  switch (mode) {
    case kApply: return run_stencil<T, kApply>(rows, N, l, s);
    case kJacobi: return run_stencil<T, kJacobi>(rows, N, l, s);
    case kJacobi2: return run_stencil<T, kJacobi2>(rows, N, l, s);
    case kResidual: return run_stencil<T, kResidual>(rows, N, l, s);
    case kNormB: return run_stencil<T, kNormB>(rows, N, l, s);
    default: return run_stencil<T, kApplyDot>(rows, N, l, s);
  }
}

template <typename T>
void run_iface(const Launch<GroupArgs<T>>& l, hipStream_t s) {
  if (l.nwg > 0) hipLaunchKernelGGL((iface_kernel<T>), dim3(l.nwg), dim3(kIfaceWG), 0, s, l);
}

template <typename T>
int dispatch(int dim, int mode, const Level& L, const void* x, void* y, const void* b, double omega, double* part,
             hipStream_t s) {
  if (mode == kDirichletSet) {
    run_iface<T>(single(iface_args<T>(L, y, b), iface_blocks(L)), s);
  } else {
    const StencilArgs<T> a = stencil_args<T>(L, x, y, b, omega, part);
    if (dim == 3) return launch_stencil3(mode, shape3(L.N).R, single(a, a.nwg), s);
    return run_stencil<T>(mode, L.rows2(dtype_of<T>()), L.N, single(a, a.nwg, L.lead2(dtype_of<T>())), s);
  }
  return check_launch();
}

int launch(const mf_mesh* m, const Level& L, int dtype, int mode, const void* x, void* y, const void* b,
           double omega, double* part, hipStream_t s) {
  return dtype == MF_F64 ? dispatch<double>(m->dim, mode, L, x, y, b, omega, part, s)
                         : dispatch<float>(m->dim, mode, L, x, y, b, omega, part, s);
}

// ---------------------------------------------------------------- batched
template <typename T>
int batch_dispatch(const BatchOp& op, const char* table, hipStream_t s) {
  if (op.kind == kOpIface) {
    run_iface<T>(batched<GroupArgs<T>>(op, table), s);
  } else if (op.dim == 3) {
    return launch_stencil3(op.mode, op.variant, batched<StencilArgs<T>>(op, table), s);
  } else {
    return run_stencil<T>(op.mode, op.variant, 0, batched<StencilArgs<T>>(op, table), s);
  }
  return check_launch();
}

}  // namespace

int64_t stencil_partials(const Level& L, int dtype) { return L.n_partials(dtype); }

int launch_stencil(const mf_mesh* m, const Level& L, int dtype, int mode, const void* x, void* y, const void* b,
                   double omega, double* part, hipStream_t s) {
  return launch(m, L, dtype, mode, x, y, b, omega, part, s);
}

int launch_iface(const mf_mesh* m, const Level& L, int dtype, int mode, const void* x, void* y, const void* b,
                 hipStream_t s) {
  return launch(m, L, dtype, mode, x, y, b, 0.0, nullptr, s);
}

int launch_exchange_apply(const Level& L, int dtype, void* y, hipStream_t s) {
  const int nblk = exchange_blocks(L);
  if (nblk == 0) return MF_OK;
  if (dtype == MF_F64)
    hipLaunchKernelGGL((exchange_kernel<double>), dim3(nblk), dim3(kIfaceWG), 0, s, exchange_args<double>(L, y));
  else
    hipLaunchKernelGGL((exchange_kernel<float>), dim3(nblk), dim3(kIfaceWG), 0, s, exchange_args<float>(L, y));
  return check_launch();
}

int launch_reduce(const double* part, int64_t np, double* result, hipStream_t s, double* copy) {
  hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(kRedT), 0, s, single(ReduceArgs{part, np, result, copy, 0, 0}, 1));
  return check_launch();
}

int launch_reduce_shift(const double* part, int64_t np, double* result, hipStream_t s) {
  hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(kRedT), 0, s, single(ReduceArgs{part, np, result, nullptr, 1, 0}, 1));
  return check_launch();
}

int launch_stencil_batch(const BatchOp& op, const char* table, hipStream_t s) {
  if (op.nwg <= 0) return MF_OK;
  if (op.kind == kOpReduce) {
    hipLaunchKernelGGL(reduce_kernel, dim3(op.nwg), dim3(kRedT), 0, s, batched<ReduceArgs>(op, table));
    return check_launch();
  }
  return op.dtype == MF_F64 ? batch_dispatch<double>(op, table, s) : batch_dispatch<float>(op, table, s);
}

}  // namespace mf

// Device code of the 3D stencil launches (gfx950): the interior walk of the
// tetrahedral macros and the macro faces.  A launch's tile list mixes these and
// the macro edges and vertices (edges.hpp), so that every row of the level,
// shared DoFs included, is finished by one launch.
#pragma once

#include <hip/hip_runtime.h>

#include "edges.hpp"
#include "rows.hpp"
#include "wave.hpp"

namespace mf {

// ------------------------------------------------------------------ buffers
// Bounds-checked accesses relative to a base: a load past the end gives 0, a
// store past it is dropped, so neither needs a clamp or a branch.  Offsets
// are bytes; kDrop is past every buffer (sizes are capped below it).
namespace buf {

using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr unsigned kDrop = 0x80000000u;

template <typename T>
__device__ __forceinline__ Rsrc make(const T* p, int64_t n) {
  // address and size are the same for all lanes, but part of their 64-bit
  // arithmetic is vector instructions: without the moves back to scalar
  // registers every access would loop over the lanes' descriptors
  const uint64_t u = (uint64_t)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)u), hi = __builtin_amdgcn_readfirstlane((int)(u >> 32));
  const int64_t bytes = n * (int64_t)sizeof(T);
  const int size = __builtin_amdgcn_readfirstlane((int)(bytes < 0x7fffffff ? bytes : 0x7fffffff));
  return __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)hi << 32 | lo), (short)0, size, 0x00027000);
}

typedef unsigned U2 __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ T ld(Rsrc r, unsigned off) {
  if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
template <typename T>
__device__ __forceinline__ void st(Rsrc r, unsigned off, T v) {
  if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, off, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, 0);
}

}  // namespace buf

// ------------------------------------------------------------------ interior
// Rows off the y = 0 and z = 0 faces, in a slab of nz slices from z0: the
// interior points, and the x = 0 and far-face (x + y + z = N) points where
// those faces are Dirichlet (they copy x), so that such rows are written
// without holes.  The slab's rows are taken in bands of R (band b: rows
// R b + 1 .. R b + R); a band's columns are those of its first row in slice z0
// (x = 0 .. N - z0 - R b - 1), so every output's x +- 1 neighbours are columns
// of the same band.  The bands' columns are numbered one after the other and
// a wave takes 64 consecutive ones (62 outputs), so that short rows fill the
// lanes as long ones do.
//
// Each lane walks its column upward through the slices with the rows
// R b .. R b + R + 1 of four slices in registers.  Storage offsets are per lane
// and advance by additions: in a slice of side S, row y + 1 starts S + 1 - y
// after row y, and (x, y, z + 1) lies T(S) - y after (x, y, z), T(S) being
// the slice's points.  Rows and slices past the macro's far face give values
// that no output uses; offsets past the macro's end are outside the buffer.
//
// Bound: memory.  Against pencils of 62 columns x 4 rows x 8 slices whose lanes
// past a row's end idled and whose boundary rows took per-lane weights from
// LDS, this needs 8.2 million wave instructions instead of 23 at N = 256 (cube,
// FP64 apply) and no second launch over shared DoFs: 94.0 -> 70.5 us per apply (3.9 TB/s of x
// and y; a copy that walks the same way runs at 4.0, a straight one at 6.1);
// two FP32 sweeps 160 -> 92 us; N = 128 FP64 apply 28 -> 10.3 us.  Rows written
// with holes (boundary points left to other tiles) cost 6 us more: a line
// that leaves the cache half written is written twice.
struct Column {
  int x, y0;  // column, row below the band's first output row
};

// q-th column of the slab of side A = N - z0: band b starts at
// b A - R b (b - 1) / 2, so b is the smaller root of
// R b^2 - (2 A + R) b + 2 q = 0, rounded down and corrected by one step either
// way (FP32: the discriminant is within an ulp and the root within an ulp).
template <int R>
__device__ __forceinline__ Column column_of(int A, int q) {
  const float c = (float)(2 * A + R);
  int b = (int)((c - __builtin_amdgcn_sqrtf(fmaxf(c * c - (float)(8 * R) * (float)q, 0.0f))) * (0.5f / R));
  auto start = [&](int k) { return k * A - R * ((k * (k - 1)) >> 1); };
  b = max(b, 0);
  if (start(b) > q) --b;
  else if (start(b + 1) <= q) ++b;
  return Column{q - start(b), R * b};
}

// What a lane writes: output (j, k) — row y0 + j, slice z0 + k, j >= 1 — where
// key + j + k < lim: interior points, and the far face's where it is
// Dirichlet; x = 0 only where that face is (off the far face).
struct WalkLane {
  Column col;
  int key, lim, A;
  bool left;
  __device__ __forceinline__ bool writes(int jk) const { return key < lim - jk; }
  // (of the points written) on the Dirichlet boundary
  __device__ __forceinline__ bool copies(int jk) const { return left || key == A - jk; }
};
template <int R>
__device__ __forceinline__ WalkLane walk_lane(const Tile& t, const MacroDev& M) {
  constexpr int kFarBit = full_mask(3) & ~1, kLeftBit = full_mask(3) & ~2;
  const int lane = threadIdx.x & (kWave - 1), q = t.x0 + lane, Q = t.y0;
  WalkLane w;
  const int N = uniform(M.N), dir_mask = uniform(M.dir_mask);
  w.A = N - (t.z & 0xffff);
  w.col = column_of<R>(w.A, min(max(q, 0), Q - 1));
  const int copy_far = (dir_mask >> kFarBit) & 1, copy_left = (dir_mask >> kLeftBit) & 1;
  w.lim = w.A + copy_far;
  w.left = w.col.x == 0;
  const bool mine = (unsigned)(lane - 1) < (unsigned)kTileW && (unsigned)q < (unsigned)Q && (!w.left || copy_left);
  w.key = mine ? w.col.x + w.col.y0 + (w.left ? copy_far : 0) : N + 1;
  return w;
}

// A column's place in the slices of its slab, from slice z0 - 1 upward.
template <typename T>
struct Cursor {
  unsigned off, row;  // bytes: offset of row y0's point from the first point of slice z0 - 1, length of row y0
  unsigned yb;
  int S;  // side of the slice
  __device__ __forceinline__ Cursor(int A, const Column& c)
      : off((unsigned)(row_start(A + 1, c.y0) + c.x) * (unsigned)sizeof(T)),
        row((unsigned)(A + 2 - c.y0) * (unsigned)sizeof(T)),
        yb((unsigned)c.y0 * (unsigned)sizeof(T)),
        S(A + 1) {}
  __device__ __forceinline__ void next() {
    off += (unsigned)(((S + 1) * (S + 2)) >> 1) * (unsigned)sizeof(T) - yb;
    row -= (unsigned)sizeof(T);
    --S;
  }
};

template <typename T, int MODE, int R>
__device__ __forceinline__ void walk3(const Tile& t, const MacroDev& M, const T* __restrict__ X, T* __restrict__ Y,
                                      const T* __restrict__ B, T omega, double& ss, double& mx) {
  using wave::dn1;
  using wave::up1;
  constexpr bool kX = MODE != kNormB;                      // reads x
  constexpr bool kB = MODE != kApply && MODE != kApplyDot;  // reads b
  constexpr bool kZ = MODE == kJacobi2;                     // as X: scaled to the iterate when its slice is first used
  constexpr unsigned E = sizeof(T);
  const int N = uniform(M.N), z0 = t.z & 0xffff, nz = t.z >> 16;
  const T* wrow = Prec<T>::row(M, full_mask(3));
  T w[15];
#pragma unroll
  for (int o = 0; o < 15; ++o) w[o] = uniform(wrow[o]);
  const T invd = kB ? uniform(Prec<T>::invd(M)) : T(0);
  const WalkLane wl = walk_lane<R>(t, M);
  const int64_t sb = uniform(M.base) + slice_base(N, z0 - 1);
  const int64_t rest = tet_count_small(N + 1) - slice_base(N, z0 - 1);
  const buf::Rsrc bx = buf::make(X + sb, rest), by = buf::make(Y + sb, rest);
  const buf::Rsrc bb = kB ? buf::make(B + sb, rest) : bx;

  Cursor<T> in(wl.A, wl.col), out(wl.A, wl.col);
  out.next();
  constexpr int NS = 4;  // slices in registers: the three an output slice reads, and the next
  T s[NS][R + 2];
  auto load_slice = [&](T* v) {
    unsigned r = in.off;
#pragma unroll
    for (int j = 0; j < R + 2; ++j) {
      v[j] = buf::ld<T>(bx, r);
      r += in.row - (unsigned)j * E;
    }
    in.next();
  };
  unsigned oq[2][R];  // offsets of the output rows
  T bq[2][R];
  auto out_rows = [&](unsigned* off, T* v) {
    unsigned r = out.off;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      r += out.row - (unsigned)j * E;
      off[j] = r;
      if (kB && !kZ) v[j] = buf::ld<T>(bb, r);
    }
    out.next();
  };
  if (kX) {
#pragma unroll
    for (int i = 0; i < NS; ++i) load_slice(s[i]);
  }
  out_rows(oq[0], bq[0]);
  // kJacobi2: omega / diagonal of the column's points inside and on the far face, of rows y > 0 and (zy) of the
  // row below the band where that is y = 0; slice i of the slab, b of the outputs kept in v
  T zi = T(0), zf = T(0), zyi = T(0), zyf = T(0);
  auto iterate_slice = [&](T* a, int i, T ci, T cf, T cyi, T cyf, T* v) {
    if (v) {
#pragma unroll
      for (int j = 1; j <= R; ++j) v[j - 1] = a[j];
    }
    const int far = wl.A + 1 - i - wl.col.x - wl.col.y0;  // its row on the far face
#pragma unroll
    for (int j = 0; j < R + 2; ++j) a[j] *= far == j ? (j == 0 ? cyf : cf) : (j == 0 ? cyi : ci);
  };
  if (kZ) {
    const int mx = wl.left ? 0 : 2, my = wl.col.y0 == 0 ? 0 : 4;
    auto c = [&](int mask) { return omega * Prec<T>::zinv(M, mask); };
    zi = c(13 | mx), zf = c(12 | mx), zyi = c(9 | mx | my), zyf = c(8 | mx | my);
    if (z0 == 1) iterate_slice(s[0], 0, c(5 | mx), c(4 | mx), c(1 | mx | my), c(mx | my), nullptr);
    else iterate_slice(s[0], 0, zi, zf, zyi, zyf, nullptr);
    iterate_slice(s[1], 1, zi, zf, zyi, zyf, bq[0]);
  }
  for (int k0 = 0; k0 < nz; k0 += NS) {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int k = k0 + i;
      if (k >= nz) break;
      out_rows(oq[(i + 1) % 2], bq[(i + 1) % 2]);
      const T* a0 = s[i];
      const T* a1 = s[(i + 1) % NS];
      if (kZ) iterate_slice(s[(i + 2) % NS], k + 2, zi, zf, zyi, zyf, bq[(i + 1) % 2]);
      const T* a2 = s[(i + 2) % NS];
#pragma unroll
      for (int j = 1; j <= R; ++j) {
        T acc = T(0);
        if (kX) {
          // the terms with dx = -1 and dx = +1 are summed in the neighbour's
          // lane and shifted once each (a shift is two moves in FP64).  The
          // point's own term, the largest, comes last: one rounding at its size
          // (FP32 apply, cube at level 5, 1.5e-8 off; with the term in its place
          // 2.3e-8, summed in the stencil's order 2.1e-8)
          T l = w[3] * a0[j + 1], r = w[1] * a0[j];
          acc = w[0] * a0[j];
          acc = fma(w[2], a0[j + 1], acc);
          acc = fma(w[4], a1[j - 1], acc);
          l = fma(w[6], a1[j], l);
          r = fma(w[5], a1[j - 1], r);
          l = fma(w[9], a1[j + 1], l);
          r = fma(w[8], a1[j], r);
          acc = fma(w[10], a1[j + 1], acc);
          l = fma(w[13], a2[j], l);
          r = fma(w[12], a2[j - 1], r);
          acc = fma(w[11], a2[j - 1], acc);
          acc = fma(w[14], a2[j], acc);
          acc = fma(w[7], a1[j], (acc + up1(l)) + dn1(r));
        }
        const T bv = bq[i % 2][j - 1], xc = a1[j];
        const bool wr = wl.writes(j + k);
        T v = row_value<T, MODE>(acc, xc, bv, omega, invd);
        v = wl.copies(j + k) ? dirichlet_row<T, MODE>(xc, bv) : v;
        if (MODE != kNormB) buf::st<T>(by, wr ? oq[i % 2][j - 1] : buf::kDrop, v);
        if (has_partials(MODE)) accum<T, MODE>(ss, mx, wr ? v : T(0), wr ? xc : T(0));
      }
      if (kX && k + NS < nz + 2) load_slice(s[i]);
    }
  }
}

// ------------------------------------------------------------------ faces
// Whether offset o of the 3D stencil stays in the macro at an inner point of
// its face f (f = 0: x + y + z = N, f = 1..3: x, y, z = 0).
__host__ __device__ constexpr bool on_side(int f, int o) {
  constexpr StencilTable ST = stencil_table(3);
  return f == 0 ? ST.off[o][0] + ST.off[o][1] + ST.off[o][2] <= 0 : ST.off[o][f - 1] >= 0;
}

// Partial row of an inner point of face F of macro M (X points at it): its 11
// neighbours in the macro, in table order.
template <typename T, int F, int MODE>
__device__ __forceinline__ T face_partial(const MacroDev& M, const T* X, int N, int x, int y, int z, T omega) {
  constexpr StencilTable ST = stencil_table(3);
  const T* w = Prec<T>::row(M, full_mask(3) & ~(1 << F));
  int off[15];
  nbr_offsets3(N, y, z, off);
  T v[15], acc = T(0);
#pragma unroll
  for (int o = 0; o < 15; ++o)
    if (on_side(F, o)) v[o] = X[off[o]];
#pragma unroll
  for (int o = 0; o < 15; ++o)
    if (on_side(F, o))
      v[o] = iterate<T, MODE>(M, support_mask(3, N, x + ST.off[o][0], y + ST.off[o][1], z + ST.off[o][2]), omega, v[o]);
#pragma unroll
  for (int o = 0; o < 15; ++o)
    if (on_side(F, o)) acc = fma(uniform(w[o]), v[o], acc);
  return acc;
}

// Storage index in copy C of the face point with weights wa, wb (and its x, y, z).
__device__ __forceinline__ int64_t face_index(const MacroDev* md, const FaceCopy& C, int N, int wa, int wb, int& x,
                                              int& y, int& z) {
  x = C.n[0] * N + C.a[0] * wa + C.b[0] * wb;
  y = C.n[1] * N + C.a[1] * wa + C.b[1] * wb;
  z = C.n[2] * N + C.a[2] * wa + C.b[2] * wb;
  return uniform(md[C.macro].base) + idx3(N, x, y, z);
}

// t.y0 inner points of the Dirichlet face t.z from its t.x0-th on (they copy
// x), four at a time per lane: their loads are issued before any store.
template <typename T, int MODE>
__device__ __forceinline__ void face_copies(const StencilArgs<T>& a, const Tile& t, double& ss, double& mx) {
  constexpr bool kX = MODE != kNormB;
  constexpr bool kB = MODE == kResidual || MODE == kNormB || MODE == kJacobi2;
  constexpr int U = 4;
  const FaceDev& F = a.faces[t.z];
  for (int i0 = threadIdx.x & (kWave - 1); i0 < t.y0; i0 += U * kWave) {
    int64_t at[U];
    T xc[U], bv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int ia, ib, x, y, z;
      slice_xy3(F.N - 3, t.x0 + min(i0 + u * kWave, t.y0 - 1), ia, ib);
      at[u] = face_index(a.md, F.cp[0], F.N, ia + 1, ib + 1, x, y, z);
      xc[u] = kX ? a.X[at[u]] : T(0);
      bv[u] = kB ? a.B[at[u]] : T(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * kWave >= t.y0) break;
      const T out = dirichlet_row<T, MODE>(xc[u], bv[u]);
      if (MODE != kNormB) a.Y[at[u]] = out;
      accum<T, MODE>(ss, mx, out, xc[u]);
    }
  }
}

// t.y0 inner points of macro face t.z (not Dirichlet) from its t.x0-th on:
// whole rows, summed over the face's one or two macros in the face's order,
// written to every copy.  Macro, face and weights are the same for all lanes
// (scalar registers), so a copy's row is 11 gathers and as many FMAs.
template <typename T, int MODE>
__device__ __forceinline__ void face_rows(const StencilArgs<T>& a, const Tile& t, double& ss, double& mx) {
  constexpr bool kX = MODE != kNormB;
  constexpr bool kB = MODE != kApply && MODE != kApplyDot;
  const FaceDev& F = a.faces[t.z];
  if (F.dirichlet) return face_copies<T, MODE>(a, t, ss, mx);
  const int N = F.N;
  for (int i = threadIdx.x & (kWave - 1); i < t.y0; i += kWave) {
    int ia, ib;
    slice_xy3(N - 3, t.x0 + i, ia, ib);
    int64_t at[2];
    int x[2], y[2], z[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) at[c] = face_index(a.md, F.cp[c], N, ia + 1, ib + 1, x[c], y[c], z[c]);
    const T bv = kB ? a.B[at[0]] : T(0);
    const T inv = sizeof(T) == 8 ? (T)F.inv : (T)F.invf;
    const T xc = MODE == kJacobi2 ? (a.omega * inv) * bv : (kX ? a.X[at[0]] : T(0));
    T acc = T(0);
    if (kX) {
      for (int c = 0; c < F.copies; ++c) {
        const MacroDev& M = a.md[F.cp[c].macro];
        const T* Xc = a.X + (c == 0 ? at[0] : at[1]);
        const int xp = c == 0 ? x[0] : x[1], yp = c == 0 ? y[0] : y[1], zp = c == 0 ? z[0] : z[1];
        switch (F.cp[c].face) {
          case 0: acc += face_partial<T, 0, MODE>(M, Xc, N, xp, yp, zp, a.omega); break;
          case 1: acc += face_partial<T, 1, MODE>(M, Xc, N, xp, yp, zp, a.omega); break;
          case 2: acc += face_partial<T, 2, MODE>(M, Xc, N, xp, yp, zp, a.omega); break;
          default: acc += face_partial<T, 3, MODE>(M, Xc, N, xp, yp, zp, a.omega); break;
        }
      }
    }
    const T out = row_value<T, MODE>(acc, xc, bv, a.omega, inv);
    if (MODE != kNormB) {
      a.Y[at[0]] = out;
      if (F.copies == 2) a.Y[at[1]] = out;
    }
    accum<T, MODE>(ss, mx, out, xc);
  }
}

}  // namespace mf

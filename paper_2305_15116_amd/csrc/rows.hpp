// Device helpers shared by the stencil, transfer and V-cycle tail kernels:
// precision-specific macro constants, the per-point partial stencil sum and
// row finish of the stencil kernels, argument resolution of batched
// launches, and the per-segment transfer and zero-iterate Jacobi steps.
#pragma once

#include <hip/hip_runtime.h>

#include "kargs.hpp"

namespace mf {

template <typename T>
struct Prec;

template <>
struct Prec<double> {
  static __device__ __forceinline__ double zinv(const MacroDev& M, int mask) { return M.zinv[mask]; }
  static __device__ __forceinline__ double w(const MacroDev& M, int mask, int i) { return M.wm[mask][i]; }
  static __device__ __forceinline__ const double* row(const MacroDev& M, int mask) { return M.wm[mask]; }
  static __device__ __forceinline__ const double& invd(const MacroDev& M) { return M.inv_diag; }
  static __device__ __forceinline__ double ginv(const double* d, const float*, int g) { return d[g]; }
  static __device__ __forceinline__ const double* K(const MacroDev& M, int t) { return M.K[t]; }
};

template <>
struct Prec<float> {
  static __device__ __forceinline__ float zinv(const MacroDev& M, int mask) { return M.zinvf[mask]; }
  static __device__ __forceinline__ float w(const MacroDev& M, int mask, int i) { return M.wmf[mask][i]; }
  static __device__ __forceinline__ const float* row(const MacroDev& M, int mask) { return M.wmf[mask]; }
  static __device__ __forceinline__ const float& invd(const MacroDev& M) { return M.inv_diagf; }
  static __device__ __forceinline__ float ginv(const double*, const float* f, int g) { return f[g]; }
  static __device__ __forceinline__ const float* K(const MacroDev& M, int t) { return M.Kf[t]; }
};

// Ordinary (write-back) stores: partial lines at wave boundaries merge in L2.
#ifndef MF_NT_STORE
#define MF_NT_STORE 0
#endif
template <typename T>
__device__ __forceinline__ void st(T* p, T v) {
  if (MF_NT_STORE) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// A macro's 16 x 16 partial-stencil table (row = support mask).  The stencil
// kernels keep a copy in LDS, so that the per-lane lookups of boundary lanes
// are LDS reads and never wait on the vector-memory counter that paces the
// row loads in flight; the V-cycle tail reads the macro record directly.
template <typename T>
using WTab = T (*)[16];

// Partial stencil sum for a point with support `mask`: neighbours outside
// the macro (whose values in v are clamped stand-ins) are dropped by
// selects, so the code is branch-free.
template <typename T, int DIM>
__device__ __forceinline__ T partial_sum(const WTab<T> W, int mask, int N, int x, int y, int z, const T* v) {
  constexpr StencilTable ST = stencil_table(DIM);
  T acc = T(0);
#pragma unroll
  for (int o = 0; o < ST.n; ++o) {
    const int nx = x + ST.off[o][0], ny = y + ST.off[o][1], nz = z + ST.off[o][2];
    const bool in = nx >= 0 && ny >= 0 && nz >= 0 && nx + ny + nz <= N;
    acc = fma(W[mask][o], in ? v[o] : T(0), acc);
  }
  return acc;
}

// Norm / dot partials of one finished row value `out` (xc = the point's x).
template <typename T, int MODE>
__device__ __forceinline__ void accum(double& ss, double& mx, T out, T xc) {
  if (MODE == kResidual || MODE == kNormB) {
    ss += (double)out * (double)out;
    mx = fmax(mx, fabs((double)out));
  } else if (MODE == kApplyDot) {
    ss += (double)xc * (double)out;  // (no maximum: only the dot product is used)
  }
}

// Finish the row of one point.  acc is its (partial) stencil value, xc and bv
// its x and b entries; it is an interior or Dirichlet point (identity row), or one
// that no other macro shares.  Norm partials count each unique DoF once
// (Dirichlet DoFs on shared primitives only in their owner).
template <typename T, int DIM, int MODE>
__device__ __forceinline__ void finish(const MacroDev& M, const WTab<T> W, int mask, T acc, T xc, T bv, T omega,
                                       T* yp, double& ss, double& mx) {
  constexpr int FM = full_mask(DIM);
  constexpr StencilTable ST = stencil_table(DIM);
  const bool full = mask == FM;
  const bool dir = !full && ((M.dir_mask >> mask) & 1);
  if (dir) {
    const T out = MODE == kResidual ? bv - xc : (MODE == kNormB ? bv : (MODE == kJacobi2 ? T(0) : xc));
    if (MODE != kNormB) st(yp, out);
    if ((M.own_mask >> mask) & 1) accum<T, MODE>(ss, mx, out, xc);
  } else {
    T out;
    if (MODE == kApply || MODE == kApplyDot) out = acc;
    else if (MODE == kJacobi || MODE == kJacobi2) out = fma(omega * (full ? Prec<T>::invd(M) : T(1) / W[mask][ST.centre]), bv - acc, xc);
    else if (MODE == kResidual) out = bv - acc;
    else out = bv;
    if (MODE != kNormB) st(yp, out);
    accum<T, MODE>(ss, mx, out, xc);
  }
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
  return v;
}

// LDS of a stencil kernel's partials
constexpr int partials_lds(int mode) { return has_partials(mode) ? 2 * kWavesPerWG * (int)sizeof(double) : 0; }

// One (sum, maximum) partial per workgroup of NW waves, summed in a fixed
// order, into slot n of part (maxima at np).  Called by every thread.
template <int NW>
__device__ __forceinline__ void wg_partial(double ss, double mx, double* part, int np, int n) {
  __shared__ double s_ss[NW], s_mx[NW];
  ss = wave_sum(ss);
  mx = wave_max(mx);
  const int wv = (int)threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    s_ss[wv] = ss;
    s_mx[wv] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double p = s_ss[0], q = s_mx[0];
#pragma unroll
    for (int k = 1; k < NW; ++k) {
      p += s_ss[k];
      q = fmax(q, s_mx[k]);
    }
    part[n] = p;
    part[np + n] = q;
  }
}

// Argument tables are read-only for the whole launch: reading them through
// the constant address space lets the compiler use scalar loads, so the
// request's arguments stay in scalar registers as a by-value argument does.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* as_const(const T* p) {
  return (const __attribute__((address_space(4))) T*)p;
}

// A record or a value of one at a wave-uniform address: a scalar load, whatever
// the compiler can prove about the kernel's stores.
template <class V>
__device__ __forceinline__ V uniform(const V& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return *as_const(&v);
#else
  return v;  // the host pass only type-checks device code
#endif
}

__device__ __forceinline__ int find_seg_c(const int32_t* wg0, int nseg, int g) {
  const auto* w = as_const(wg0);
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (w[mid] <= g) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Resolves workgroup g of a launch to its request's arguments and the
// workgroup index inside that request.
template <class A>
__device__ __forceinline__ int resolve(const Launch<A>& L, int g, A& a) {
  if (L.nseg == 0) {
    a = L.one;
    return g;
  }
  const int r = find_seg_c(L.wg0, L.nseg, g);
#if defined(__HIP_DEVICE_COMPILE__)
  a = as_const(L.many)[r];
#else
  a = L.many[r];  // the host pass only type-checks device code
#endif
  return g - as_const(L.wg0)[r];
}

template <int DIM>
__device__ __forceinline__ int64_t lidx(int N, int x, int y, int z) {
  return DIM == 2 ? idx2(N, x, y) : idx3(N, x, y, z);
}

// Segment and macro records are read-only for the launch: read them through
// the constant address space (scalar loads, scalar registers).
__device__ __forceinline__ Tile load_seg(const Tile* segs, int si) {
#if defined(__HIP_DEVICE_COMPILE__)
  return as_const(segs)[si];
#else
  return segs[si];
#endif
}

struct MacroC {
  int64_t base;
  int32_t N;
  uint16_t own_mask, dir_mask, shared_mask;
};

__device__ __forceinline__ MacroC load_macro(const MacroDev* md, int m) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto* p = as_const(md) + m;
  return MacroC{p->base, p->N, p->own_mask, p->dir_mask, p->shared_mask};
#else
  return MacroC{md[m].base, md[m].N, md[m].own_mask, md[m].dir_mask, md[m].shared_mask};
#endif
}

// Storage offsets of the 15 stencil neighbours of a 3D point (x, y, z),
// relative to the point, in stencil-table order; exact for neighbours inside
// the macro.  Slice z has side S = N - z and row y of it d = S + 1 - y
// points: rows y +- 1 start d after / end d + 1 before the point's column,
// and (x, y, z + 1) / (x, y, z - 1) lie T(S) - y after / T(S + 1) - y
// before it (T(s) = (s + 1)(s + 2) / 2 points in a slice of side s).
__device__ __forceinline__ void nbr_offsets3(int N, int y, int z, int (&o)[15]) {
  const int S = N - z, d = S + 1 - y;
  const int up = (S + 1) * (S + 2) / 2 - y;
  const int dn = y - (S + 2) * (S + 3) / 2;
  const int t[15] = {dn, dn + 1, dn + d + 1, dn + d, -d - 1, -d, -1, 0, 1, d - 1, d, up - d, up - d + 1, up - 1, up};
#pragma unroll
  for (int k = 0; k < 15; ++k) o[k] = t[k];
}

// Restriction r_c = P^T r_f on one macro: a coarse point P gathers the fine
// point 2P (weight 1) and the fine points 2P + d for the stencil offsets d
// (weight 1/2) — the fine points whose interpolation uses P — counting only
// fine points this macro owns, so that the sum over the copies of P takes each fine DoF
// once.  Dirichlet fine points are skipped.
template <typename T, int DIM>
__device__ __forceinline__ T restrict_partial(const TransferArgs<T>& a, int macro, int x, int y, int z) {
  constexpr StencilTable ST = stencil_table(DIM);
  constexpr int full = full_mask(DIM);
  const MacroDev& F = a.mdf[macro];
  const int Nf = F.N, own = F.own_mask & ~F.dir_mask;
  int off[15];
  if constexpr (DIM == 3) nbr_offsets3(Nf, 2 * y, 2 * z, off);
  const T* p = a.src + F.base + lidx<DIM>(Nf, 2 * x, 2 * y, 2 * z);
  T acc = T(0);
#pragma unroll
  for (int s = 0; s < ST.n; ++s) {
    const int dx = ST.off[s][0], dy = ST.off[s][1], dz = ST.off[s][2];
    const int fx = 2 * x + dx, fy = 2 * y + dy, fz = 2 * z + dz;
    const bool in = fx >= 0 && fy >= 0 && fz >= 0 && fx + fy + fz <= Nf;
    const int mask = support_mask(DIM, Nf, fx, fy, fz);
    const bool use = in && (mask == full || ((own >> mask) & 1));
    const int l = Nf + 1 - 2 * y;  // 2D: the row's length
    const int o = DIM == 3 ? off[s] : dx + (dy > 0 ? l : dy < 0 ? -l - 1 : 0);
    const T r = p[in ? o : 0];
    acc += use ? (s == ST.centre ? T(1) : T(0.5)) * r : T(0);
  }
  return acc;
}
// (x, y) of slice-local index r in a 3D slice of side S <= 2048, r <
// (S+1)(S+2)/2: y is the smaller root of y^2 - (2S + 3) y + 2r = 0 (row y
// starts at y (2S + 3 - y) / 2), rounded down and corrected by one step
// either way.  The FP32 discriminant is exact or within an ulp and the
// hardware root within an ulp, far inside that correction.
__device__ __forceinline__ void slice_xy3(int S, int r, int& x, int& y) {
  const float b = 2.0f * (float)S + 3.0f;
  int yy = (int)((b - __builtin_amdgcn_sqrtf(b * b - 8.0f * (float)r)) * 0.5f);
  yy = min(max(yy, 0), S);
  if (row_start(S, yy) > r) --yy;
  else if (yy < S && row_start(S, yy + 1) <= r) ++yy;
  y = yy;
  x = r - row_start(S, yy);
}

// The same in either dimension: slice index r < (S + 1)(S + 2) / 2 of a slice of
// side S (2D: the macro).
template <int DIM>
__device__ __forceinline__ void slice_xy(int S, int r, int& x, int& y) {
  if (DIM == 3) {
    slice_xy3(S, r, x, y);
    return;
  }
  // 2D: the discriminant reaches 2^32, exact in a double
  const double b = 2.0 * (double)S + 3.0;
  int yy = (int)((b - sqrt(b * b - 8.0 * (double)r)) * 0.5);
  yy = min(max(yy, 0), S);
  if (row_start(S, yy) > r) --yy;
  else if (yy < S && row_start(S, yy + 1) <= r) ++yy;
  y = yy;
  x = r - row_start(S, yy);
}
// Restriction by segments of 64 coarse points: restrict_partial's sum, in its
// order, for a lane's point P.  The fine points come in neighbouring pairs (8
// or 16 bytes) of the rows around 2P: x and x + 1 where dx is 0 or 1, x - 1 and
// x where it is -1 or 0.  Whether 2P + d lies in the macro, and its support,
// follow from P's position: 2x + dx = 0 only for x = 0 and dx = 0, and N_f -
// |2P + d| = 2 (N_c - |P|) - |d| vanishes only on P's far face with |d| = 0.
// Rows outside the macro read the point itself.  load() issues every load,
// store() sums and writes: 0 at Dirichlet points, nothing at shared ones (without
// boundary tiles, nb = 0: the macro's part).
template <typename T, int DIM>
struct RestrictCell {
  typedef T Pair __attribute__((ext_vector_type(2), aligned(sizeof(T))));
  bool live, x0, y0, z0, far, first, parts;
  int own, mask, out;  // out: the coarse point's masks (dir, shared) as bits 0, 1
  T* at;
  Pair A, B, Cc, D, E, Ff, G;
  T xp;

  __device__ __forceinline__ void load(const TransferArgs<T>& a, const Tile& sg) {
    const MacroC C = load_macro(a.mdc, sg.macro);
    const MacroC F = load_macro(a.mdf, sg.macro);
    const int z = DIM == 3 ? sg.z : 0, S = C.N - z, P = (S + 1) * (S + 2) / 2;
    parts = a.nb == 0;
    int r = sg.x0 + (int)(threadIdx.x & (kWave - 1)), x, y;
    live = r < P;
    r = min(r, P - 1);
    slice_xy<DIM>(S, r, x, y);
    x0 = x == 0, y0 = y == 0, z0 = DIM == 2 || z == 0, far = x + y == S;
    own = F.own_mask & ~F.dir_mask;
    mask = (far ? 0 : 1) | (x0 ? 0 : 2) | (y0 ? 0 : 4) | (DIM == 2 || z0 ? 0 : 8);
    const bool full = mask == full_mask(DIM);
    out = full ? 0 : ((C.dir_mask >> mask) & 1) | (((C.shared_mask >> mask) & 1) << 1);
    at = a.dst + C.base + (DIM == 3 ? as_const(a.sbc)[z] : 0) + r;
    // offsets from the first point of fine slice 2z - 1 (of slice 0 at z = 0)
    const int zf = 2 * z, za = DIM == 3 && zf > 0 ? zf - 1 : 0, Sf = F.N - zf, yf = 2 * y;
    const T* f = a.src + F.base + (DIM == 3 ? as_const(a.sbf)[za] : 0);
    const int tb = DIM == 3 ? as_const(a.sbf)[zf] - as_const(a.sbf)[za] : 0;
    const int c = tb + row_start(Sf, yf) + 2 * x, l = Sf + 1 - yf;
    auto pair = [&](bool in, int i) { return *(const Pair*)(f + (unsigned)(in ? i : max(c - 1, 0))); };
    first = x0 && !far;  // D starts at 2P
    D = *(const Pair*)(f + (unsigned)(first ? c : c - 1));
    xp = f[(unsigned)(far ? c : c + 1)];
    Cc = pair(!y0, c - l - 1);
    E = pair(!(far && x0), c + l - 1);
    if constexpr (DIM == 3) {
      const int dn = c - tb + yf, up = c + (Sf + 1) * (Sf + 2) / 2 - yf;
      A = pair(!z0, dn);
      B = pair(!z0, dn + l);
      Ff = pair(!y0, up - l);
      G = pair(!(far && x0), up - 1);
    }
  }

  __device__ __forceinline__ void store() const {
    constexpr StencilTable ST = stencil_table(DIM);
    T v[ST.n];
    const T xc = first ? D.x : D.y;
    if constexpr (DIM == 3) {
      const T t[15] = {A.x, A.y, B.y, B.x, Cc.x, Cc.y, D.x, xc, xp, E.x, E.y, Ff.x, Ff.y, G.x, G.y};
#pragma unroll
      for (int s = 0; s < ST.n; ++s) v[s] = t[s];
    } else {
      const T t[7] = {Cc.x, Cc.y, D.x, xc, xp, E.x, E.y};
#pragma unroll
      for (int s = 0; s < ST.n; ++s) v[s] = t[s];
    }
    T acc = T(0);
#pragma unroll
    for (int s = 0; s < ST.n; ++s) {
      const int dx = ST.off[s][0], dy = ST.off[s][1], dz = ST.off[s][2], sd = dx + dy + dz;
      const bool in = (dx >= 0 || !x0) && (dy >= 0 || !y0) && (dz >= 0 || !z0) && (sd <= 0 || !far);
      const int m = ((sd == 0 && far) ? 0 : 1) | ((dx == 0 && x0) ? 0 : 2) | ((dy == 0 && y0) ? 0 : 4) |
                    (DIM == 2 || (dz == 0 && z0) ? 0 : 8);
      const bool use = in && (m == full_mask(DIM) || ((own >> m) & 1));
      acc += use ? (s == ST.centre ? T(1) : T(0.5)) * v[s] : T(0);
    }
    if (live && (parts || (out & 3) != 2)) *at = out & 1 ? T(0) : acc;
  }
};

// x_f += P e_c: even fine points take the coarse value, the others the mean of
// the two coarse endpoints of the coarse micro-edge they bisect.  Its direction
// is the point's parities, with the middle odd coordinate negated for two or
// three odd ones ((1,1,0): e1 - e2, (1,0,1): e1 - e3, (0,1,1): e2 - e3, (1,1,1): e1
// - e2 + e3).  Dirichlet points are left unchanged.
//
// Prolongation by cells: a lane takes coarse point P = (X, Y, Z) and the fine
// points 2P + p, p in {0, 1}^DIM, that lie in the macro, two neighbours along x
// at a time (8 or 16 bytes, consecutive lanes consecutive pairs).  Their
// values need P and its neighbours along x, y, z and x + z; with room = N_c - |P|,
// 2P + p is in the macro if |p| <= 2 room.  load() issues every load, store()
// adds and writes; Dirichlet points are written back as they were.
template <typename T, int DIM>
struct ProlongCell {
  typedef T Pair __attribute__((ext_vector_type(2), aligned(sizeof(T))));
  static constexpr int NP = 1 << (DIM - 1);  // pairs (y, z parities)
  int room, X, Y, Z, dir;
  bool live, apex;
  T c, cx, cy, cz, cxz;
  T* at[NP];
  Pair old[NP];

  __device__ __forceinline__ void load(const TransferArgs<T>& a, const Tile& sg) {
    const MacroC C = load_macro(a.mdc, sg.macro);
    const MacroC F = load_macro(a.mdf, sg.macro);
    Z = DIM == 3 ? sg.z : 0;
    const int S = C.N - Z, P = (S + 1) * (S + 2) / 2;
    int r = sg.x0 + (int)(threadIdx.x & (kWave - 1));
    live = r < P;
    r = min(r, P - 1);
    slice_xy<DIM>(S, r, X, Y);
    room = S - X - Y;
    dir = F.dir_mask & ~(1 << full_mask(DIM));
    const T* p = a.src + C.base + (DIM == 3 ? as_const(a.sbc)[Z] : 0) + r;
    const int l = S + 1 - Y, up = (S + 1) * (S + 2) / 2 - Y;
    c = p[0];
    cx = p[room >= 1 ? 1 : 0];
    cy = p[room >= 1 ? l : 0];
    if constexpr (DIM == 3) {
      cz = p[room >= 1 ? up : 0];
      cxz = p[room >= 2 ? up + 1 : 0];
    }
    const int Sf = 2 * S, lf = Sf + 1 - 2 * Y, uf = (Sf + 1) * (Sf + 2) / 2 - 2 * Y;
    T* f = a.dst + F.base + (DIM == 3 ? as_const(a.sbf)[2 * Z] : 0) + row_start(Sf, 2 * Y) + 2 * X;
    // the macro's last point has no successor: the pair from its predecessor on
    apex = room == 0 && (DIM == 3 ? Z : Y) == C.N;
    at[0] = f;
    at[1] = f + (room >= 1 ? lf : 0);
    if constexpr (DIM == 3) {
      at[2] = f + (room >= 1 ? uf : 0);
      at[3] = f + (room >= 1 ? uf + lf - 1 : 0);
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) old[k] = *(const Pair*)(at[k] - (apex ? 1 : 0));
  }

  __device__ __forceinline__ void store() const {
    T add[NP][2] = {};
    add[0][0] = T(0.5) * (c + c);
    add[0][1] = T(0.5) * (c + cx);
    add[1][0] = T(0.5) * (c + cy);
    add[1][1] = T(0.5) * (cy + cx);
    if constexpr (DIM == 3) {
      add[2][0] = T(0.5) * (c + cz);
      add[2][1] = T(0.5) * (cz + cx);
      add[3][0] = T(0.5) * (cz + cy);
      add[3][1] = T(0.5) * (cy + cxz);
    }
    const bool edge = X == 0 || Y == 0 || (DIM == 3 && Z == 0) || room <= 1;
    bool keep[NP][2] = {};
    if (dir != 0 && __builtin_amdgcn_ballot_w64(edge)) {
#pragma unroll
      for (int k = 0; k < NP; ++k)
#pragma unroll
        for (int px = 0; px < 2; ++px) {
          const int py = k & 1, pz = k >> 1;
          const int mask = (2 * room != px + py + pz ? 1 : 0) | (X != 0 || px ? 2 : 0) | (Y != 0 || py ? 4 : 0) |
                           (DIM == 3 && (Z != 0 || pz) ? 8 : 0);
          keep[k][px] = (dir >> mask) & 1;
        }
    }
    if (!live) return;
    Pair v[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      v[k].x = apex ? old[k].y : old[k].x;
      v[k].y = old[k].y;
      if (!keep[k][0]) v[k].x += add[k][0];
      if (!keep[k][1]) v[k].y += add[k][1];
    }
    if (room == 0) {
      *at[0] = v[0].x;
      return;
    }
#pragma unroll
    for (int k = 0; k < NP - 1; ++k) *(Pair*)at[k] = v[k];
    // |p| = DIM: outside the macro for room = 1 in 3D
    if (DIM == 3 && room == 1) *at[NP - 1] = v[NP - 1].x;
    else *(Pair*)at[NP - 1] = v[NP - 1];
  }
};

// First Jacobi sweep of a V-cycle level.  The iterate is zero there, so
// x' = x + omega D^-1 (b - A x) reduces to omega D^-1 b, with D the diagonal
// of the row the sweep would finish: the macro's interior centre weight, the
// partial stencil's centre at a boundary point no other macro shares, the
// assembled diagonal of a shared DoF (exchange list), and x' = x = 0 at
// Dirichlet DoFs.  The arithmetic is that of the stencil kernels with x = 0
// (fma(omega d, b - 0, 0)), in passes that read b once.
template <typename T>
__device__ __forceinline__ T centre_inv(const MacroDev& M, int mask, int full, int centre) {
  if constexpr (sizeof(T) == 8) return mask == full ? M.inv_diag : 1.0 / M.wm[mask][centre];
  else return mask == full ? M.inv_diagf : 1.0f / M.wmf[mask][centre];
}

template <int DIM>
__device__ __forceinline__ int64_t copy_index(const MacroDev& M, const Copy& c) {
  return M.base + (DIM == 2 ? idx2(M.N, c.x, c.y) : idx3(M.N, c.x, c.y, c.z));
}

// One DoF shared by several macros and not Dirichlet (exchange list): its
// copies in Y hold partial rows; sum them in fixed macro order and write the
// row to every copy.
template <typename T>
__device__ __forceinline__ void exchange_row(const GroupArgs<T>& a, int g) {
  const int c0 = a.gptr[g], c1 = a.gptr[g + 1];
  T acc = T(0);
  for (int c = c0; c < c1; ++c) acc += a.Y[a.cidx[c]];
  for (int c = c0; c < c1; ++c) a.Y[a.cidx[c]] = acc;
}

// Coarse direct solve, unknown i, one wavefront (lane = its lane):
// x(copies of i) = sum_j Ainv[i][j] b(first copy of j).
template <typename T>
__device__ __forceinline__ void coarse_row(const CoarseArgs<T>& a, int i, int lane) {
  T acc = T(0);
  for (int j = lane; j < a.n; j += kWave) acc = fma(a.Ainv[(int64_t)i * a.n + j], a.B[a.first[j]], acc);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, kWave);
  for (int c = a.cptr[i] + lane; c < a.cptr[i + 1]; c += kWave) a.X[a.cidx[c]] = acc;
}

// The zero-iterate Jacobi row of shared non-Dirichlet DoF g (exchange list),
// written to every copy.
template <typename T, int DIM>
__device__ __forceinline__ void jacobi0_group(const Jacobi0Args<T>& a, int g) {
  const int c0 = a.gptr[g], c1 = a.gptr[g + 1];
  const T b = a.B[a.gidx[c0]];
  T d;
  if constexpr (sizeof(T) == 8) d = a.ginv[g];
  else d = a.ginvf[g];
  const T out = fma(a.omega * d, b, T(0));
  for (int c = c0; c < c1; ++c) a.Y[a.gidx[c]] = out;
}

}  // namespace mf

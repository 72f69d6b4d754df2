// The bottom of a V-cycle in one workgroup (gfx950).
//
// Below a few thousand points per level, every step of the cycle (stencil
// pass, transfer, coarse solve) takes about the same time whatever its size: a
// chain of dependent loads plus the launch, seven launches per level and
// cycle.  vcycle_tail_kernel runs the coarse solve and the levels just above
// it (kargs.hpp: kTailLevels, kTailMaxPoints) with one workgroup of 16 waves
// and a barrier between steps, the levels' vectors in LDS where they fit.  The
// steps and their order are those of the multi-launch cycle, and so is every
// point's arithmetic up to the order of the sums at DoFs shared by macros and
// the rounding of reciprocal diagonals there.
//
// What a step needs to know of a point (its lattice point, neighbours inside
// the macro, support) and of a shared DoF (where its copies are) is worked out
// once per level and kept in registers, so that a step waits for LDS and one
// table row, not for chains of global loads.  Bound: the chain of steps, about
// 1.6 us for a sweep of 1,000 points (index arithmetic and the rows' 64
// bytes per point on one CU).  FP32: six tets (990 points) 29 -> 23 us,
// nine 36 -> 26, three triangles 56 -> 44, 22 triangles 67 -> 46.
//
// One workgroup per request: a batched launch gives each member its own.

#include <hip/hip_runtime.h>

#include "launch.hpp"
#include "rows.hpp"

namespace mf {

namespace {

constexpr int kTailWaves = kTailWG / kWave;

int check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(MF_EDEVICE, hipGetErrorString(e));
  return MF_OK;
}

// A level's vectors: LDS (address space 3, so that accesses are LDS
// instructions) or global memory.
template <typename T, bool LDS>
struct TailPtr {
  typedef T* type;
};
template <typename T>
struct TailPtr<T, true> {
  typedef __attribute__((address_space(3))) T* type;
};

// Storage index of a lattice point in its macro (tail levels are small: 32 bits).
template <int DIM>
__device__ __forceinline__ int tidx(int N, int x, int y, int z) {
  return (int)lidx<DIM>(N, x, y, z);
}

// Storage offsets of a point's stencil neighbours inside its macro.
template <int DIM>
__device__ __forceinline__ void tail_offsets(int N, int y, int z, int (&off)[15]) {
  if constexpr (DIM == 3) {
    nbr_offsets3(N, y, z, off);
  } else {
    constexpr StencilTable ST = stencil_table(2);
    const int l = N + 1 - y;
#pragma unroll
    for (int o = 0; o < ST.n; ++o) off[o] = ST.off[o][0] + (ST.off[o][1] > 0 ? l : ST.off[o][1] < 0 ? -l - 1 : 0);
  }
}

// v, as a value the compiler cannot trace: what is computed from it is computed
// anew in each step, not kept in registers (spilled) between steps.
__device__ __forceinline__ int fresh(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
  return v;
}

// One row of a partial-stencil table (aligned to its elements only).
template <typename T>
__device__ __forceinline__ void load_row(const T* w, T (&r)[16]) {
  typedef T Quad __attribute__((ext_vector_type(4), aligned(sizeof(T))));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const Quad v = ((const Quad*)w)[q];
    r[4 * q] = v.x, r[4 * q + 1] = v.y, r[4 * q + 2] = v.z, r[4 * q + 3] = v.w;
  }
}

// What a thread keeps of a level for all its steps: its storage points t, t +
// kTailWG, ... (the level's points, packed: its row segments would leave most
// lanes idle in 3D) with lattice point, support, neighbours inside the macro
// and 1 / assembled diagonal (0: Dirichlet), and its DoFs shared by macros
// (exchange list) with their first copies.
template <typename T, int DIM>
struct TailState {
  static constexpr int K = (int)((kTailMaxPoints + kTailWG - 1) / kTailWG), G = (K + 1) / 2, C = sizeof(T) == 8 ? 2 : 4;
  int N, n, ng;
  const MacroDev* md;
  const int64_t* cidx;
  int xyz[K], in[K], mm[K];  // x, y, z in 10 bits each; neighbour bits; macro, mask in the low 4 bits
  bool dir[K], shared[K];
  T inv[K];
  int c0[G], nc[G], ci[G][C];
  T ginv[G];

  __device__ __forceinline__ int point(int k) const { return (int)threadIdx.x + k * kTailWG; }
  __device__ __forceinline__ bool live(int k) const { return point(k) < n; }
  __device__ __forceinline__ void lattice(int k, int& x, int& y, int& z) const {
    const int q = fresh(xyz[k]);
    x = q & 1023, y = (q >> 10) & 1023, z = q >> 20;
  }

  __device__ __forceinline__ void load(const TailLevel<T>& F) {
    constexpr StencilTable ST = stencil_table(DIM);
    N = F.N;
    md = F.md;
    cidx = F.xcidx;
    const int P = (int)macro_points(DIM, N);
    n = P * F.nmac;
    ng = F.nx;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      c0[g] = nc[g] = 0;
      const int gi = (int)threadIdx.x + g * kTailWG;
      if (gi >= ng) continue;
      c0[g] = F.xptr[gi];
      nc[g] = F.xptr[gi + 1] - c0[g];
#pragma unroll
      for (int c = 0; c < C; ++c) ci[g][c] = (int)cidx[c0[g] + min(c, nc[g] - 1)];
      ginv[g] = Prec<T>::ginv(F.xinv, F.xinvf, gi);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (k * kTailWG >= n) break;
      if (!live(k)) continue;
      const int m = point(k) / P;
      int r = point(k) - m * P, x, y = 0, z = 0, S = N;
      if (DIM == 3) {
        // slice z holds (S + 1)(S + 2) / 2 points, S = N - z
        for (int sz = (S + 1) * (S + 2) / 2; r >= sz; sz = (S + 1) * (S + 2) / 2) {
          r -= sz;
          --S;
          ++z;
        }
        slice_xy3(S, r, x, y);
      } else {
        for (int len = S + 1; r >= len; --len) {  // row y holds S + 1 - y points
          r -= len;
          ++y;
        }
        x = r;
      }
      xyz[k] = x | y << 10 | z << 20;
      const int mask = support_mask(DIM, N, x, y, z);
      mm[k] = m << 4 | mask;
      in[k] = 0;
#pragma unroll
      for (int o = 0; o < ST.n; ++o) {
        const int nx = x + ST.off[o][0], ny = y + ST.off[o][1], nz = z + ST.off[o][2];
        in[k] |= (nx >= 0 && ny >= 0 && nz >= 0 && nx + ny + nz <= N ? 1 : 0) << o;
      }
      const bool bnd = mask != full_mask(DIM);
      dir[k] = bnd && ((md[m].dir_mask >> mask) & 1);
      shared[k] = bnd && !dir[k] && ((md[m].shared_mask >> mask) & 1);
      inv[k] = Prec<T>::zinv(md[m], mask);
    }
  }

  // Sums of the copies of shared DoFs, whose partial rows are in Y: finished
  // (kApply: the sum itself) and written to every copy.
  template <int MODE, class V>
  __device__ __forceinline__ void exchange(V X, V Y, V B, T omega) const {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (g * kTailWG >= ng) break;
      if (nc[g] == 0) continue;
      T p[C], acc = T(0);
#pragma unroll
      for (int c = 0; c < C; ++c) p[c] = Y[ci[g][c]];
      const T bv = MODE != kApply ? B[ci[g][0]] : T(0), xc = MODE == kJacobi ? X[ci[g][0]] : T(0);
#pragma unroll
      for (int c = 0; c < C; ++c) acc += c < nc[g] ? p[c] : T(0);
      for (int c = C; c < nc[g]; ++c) acc += Y[(int)cidx[c0[g] + c]];
      const T out = MODE == kApply ? acc : (MODE == kJacobi ? fma(omega * ginv[g], bv - acc, xc) : bv - acc);
#pragma unroll
      for (int c = 0; c < C; ++c) Y[ci[g][c]] = out;  // (the last one again where there are fewer)
      for (int c = C; c < nc[g]; ++c) Y[(int)cidx[c0[g] + c]] = out;
    }
    __syncthreads();
  }

  // One pass over the level: Jacobi sweep or residual, Y from X and B.
  template <int MODE, class V>
  __device__ __forceinline__ void pass(V X, V Y, V B, T omega) const {
    constexpr StencilTable ST = stencil_table(DIM);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (k * kTailWG >= n) break;
      if (!live(k)) continue;
      const int i = point(k);
      int x, y, z, off[15];
      lattice(k, x, y, z);
      tail_offsets<DIM>(N, y, z, off);
      T w[16], v[ST.n];
      const int q = fresh(mm[k]), inside = fresh(in[k]);
      load_row<T>(Prec<T>::row(md[q >> 4], q & 15), w);
      // neighbours outside the macro have weight 0 and read the point itself
#pragma unroll
      for (int o = 0; o < ST.n; ++o) v[o] = X[i + ((inside >> o) & 1 ? off[o] : 0)];
      const T bv = B[i], xc = v[ST.centre];
      T acc = T(0);
#pragma unroll
      for (int o = 0; o < ST.n; ++o) acc = fma(w[o], v[o], acc);
      T out;
      if (MODE == kJacobi) out = dir[k] ? xc : (shared[k] ? acc : fma(omega * inv[k], bv - acc, xc));
      else out = dir[k] ? bv - xc : (shared[k] ? acc : bv - acc);
      Y[i] = out;
      __builtin_amdgcn_sched_barrier(0);  // one point's values in registers at a time
    }
    __syncthreads();
    if (ng > 0) exchange<MODE>(X, Y, B, omega);
  }

  // First sweep from a zero iterate.
  template <class V>
  __device__ __forceinline__ void sweep0(V Y, V B, T omega) const {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (k * kTailWG >= n) break;
      if (live(k)) Y[point(k)] = dir[k] ? T(0) : (omega * inv[k]) * B[point(k)];
    }
    __syncthreads();
  }

  template <class V>
  __device__ __forceinline__ void copy(V Y, V X) const {
    for (int i = (int)threadIdx.x; i < n; i += kTailWG) Y[i] = X[i];
    __syncthreads();
  }

  // `sweeps` Jacobi sweeps ping-ponging x <-> t, as jacobi_sweeps does; from
  // zero, the first is omega D^-1 b into t.
  template <class V>
  __device__ __forceinline__ void jacobi(V X, V Tm, V B, int sweeps, T omega, bool from_zero) const {
    if (from_zero && sweeps == 0) {
      for (int i = (int)threadIdx.x; i < n; i += kTailWG) X[i] = T(0);
      __syncthreads();
      return;
    }
    V cur = X, oth = Tm;
    int i = 0;
    if (from_zero) {
      sweep0(Tm, B, omega);
      cur = Tm, oth = X;
      i = 1;
    }
    for (; i < sweeps; ++i) {
      pass<kJacobi>(cur, oth, B, omega);
      const V s = cur;
      cur = oth;
      oth = s;
    }
    if (cur != X) copy(X, cur);
  }

  // Right-hand side of this level from the finer one's residual R: a point
  // gathers the fine points whose interpolation uses it, each counted in the
  // macro that owns it; shared DoFs sum their copies, Dirichlet ones are 0.
  template <class V>
  __device__ __forceinline__ void restrict_from(int Nf, V R, V B) const {
    constexpr StencilTable ST = stencil_table(DIM);
    constexpr int full = full_mask(DIM);
    const int Pf = (int)macro_points(DIM, Nf);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (k * kTailWG >= n) break;
      if (!live(k)) continue;
      int x, y, z, off[15];
      lattice(k, x, y, z);
      tail_offsets<DIM>(Nf, 2 * y, 2 * z, off);
      const int m = mm[k] >> 4, f = m * Pf + tidx<DIM>(Nf, 2 * x, 2 * y, 2 * z);
      const int own = md[m].own_mask, dm = md[m].dir_mask;
      T acc = T(0);
#pragma unroll
      for (int o = 0; o < ST.n; ++o) {
        const int fx = 2 * x + ST.off[o][0], fy = 2 * y + ST.off[o][1], fz = 2 * z + ST.off[o][2];
        const bool inside = fx >= 0 && fy >= 0 && fz >= 0 && fx + fy + fz <= Nf;
        const int mask = support_mask(DIM, Nf, fx, fy, fz);
        const bool use = inside && (mask == full || (((own & ~dm) >> mask) & 1));
        const T r = R[f + (inside ? off[o] : 0)];
        const T w = o == ST.centre ? T(1) : T(0.5);
        acc += use ? w * r : T(0);
      }
      B[point(k)] = dir[k] ? T(0) : acc;
    }
    __syncthreads();
    if (ng > 0) exchange<kApply>(B, B, B, T(0));
  }

  // X += the interpolation of the coarser level's E.
  template <class V>
  __device__ __forceinline__ void prolong_from(int Nc, V E, V X) const {
    const int Pc = (int)macro_points(DIM, Nc);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (k * kTailWG >= n) break;
      if (!live(k)) continue;
      int x, y, z;
      lattice(k, x, y, z);
      // direction of the coarse micro-edge the point bisects (rows.hpp)
      const int px = x & 1, py = y & 1, pz = z & 1;
      const int sx = px, sy = (px && py) ? -1 : py, sz = (pz && (px ^ py)) ? -1 : pz;
      const int c = (mm[k] >> 4) * Pc;
      const T u = E[c + tidx<DIM>(Nc, (x - sx) >> 1, (y - sy) >> 1, (z - sz) >> 1)];
      const T v = E[c + tidx<DIM>(Nc, (x + sx) >> 1, (y + sy) >> 1, (z + sz) >> 1)];
      if (!dir[k]) X[point(k)] += T(0.5) * (u + v);
    }
    __syncthreads();
  }
};

// The request's record, read in place (constant address space: scalar
// loads) rather than copied, so that the per-level records indexed by a
// loop counter need no private memory.
template <class A>
__device__ __forceinline__ auto resolve_ref(const Launch<A>& L, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (L.nseg == 0) return as_const(&L.one);
  return as_const(L.many) + find_seg_c(L.wg0, L.nseg, g);
#else
  (void)g;
  return L.nseg == 0 ? &L.one : L.many;  // the host pass only type-checks device code
#endif
}

extern __shared__ __align__(16) unsigned char tail_lds[];

template <typename T, int DIM, bool LDS, class A>
__device__ __forceinline__ void tail_cycle(const A* a) {
  using V = typename TailPtr<T, LDS>::type;
  const int nlev = a->nlev, pre = a->pre, post = a->post;
  const T omega = a->omega;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = (int)threadIdx.x & (kWave - 1);
  // Level k's b, x and t (w = 0, 1, 2).  In LDS only the top level's b comes in
  // from global memory and its x goes out.
  auto vec = [&](int k, int w) -> V {
    if constexpr (LDS) {
      int64_t off = 0;
      for (int j = 0; j < k; ++j) off += 3 * tail_lds_vec(a->lv[j].storage, (int)sizeof(T));
      return (V)(tail_lds + off + w * tail_lds_vec(a->lv[k].storage, (int)sizeof(T)));
    } else {
      return w == 0 ? a->lv[k].b : (w == 1 ? a->lv[k].x : a->lv[k].t);
    }
  };
  if constexpr (LDS) {
    const V b = vec(nlev - 1, 0);
    const T* g = a->lv[nlev - 1].b;
    for (int i = (int)threadIdx.x; i < (int)a->lv[nlev - 1].storage; i += kTailWG) b[i] = g[i];
  }
  TailState<T, DIM> F;
  F.load(a->lv[nlev - 1]);
  __syncthreads();
  // descent: levels lc + nlev - 1 .. lc + 1
  for (int k = nlev - 1; k >= 1; --k) {
    F.jacobi(vec(k, 1), vec(k, 2), vec(k, 0), pre, omega, true);
    F.template pass<kResidual>(vec(k, 1), vec(k, 2), vec(k, 0), T(0));
    F.load(a->lv[k - 1]);
    F.restrict_from(a->lv[k].N, vec(k, 2), vec(k - 1, 0));
  }
  // coarse level: x = 0, then the dense solve on its unknowns (a wave each)
  {
    const V x = vec(0, 1), b = vec(0, 0);
    for (int i = (int)threadIdx.x; i < (int)a->lv[0].storage; i += kTailWG) x[i] = T(0);
    __syncthreads();
    // b at this lane's columns, then U rows at a time (one after the other:
    // 12 us for 22 triangles, now 7)
    const int n = a->coarse.n;
    constexpr int J = kTailMaxCoarse / kWave, U = 4;
    T bj[J];
#pragma unroll
    for (int q = 0; q < J; ++q) {
      const int j = lane + q * kWave;
      bj[q] = j < n ? b[a->coarse.first[j]] : T(0);
    }
    for (int i0 = wave; i0 < n; i0 += U * kTailWaves) {
      // (loads without branches, so that all are in flight together; lanes past
      // the row's end read its last entry, times 0)
      T acc[U], av[U][J];
      int c0[U], c1[U], at[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * kTailWaves;
        if (i >= n) break;
        c0[u] = a->coarse.cptr[i] + lane, c1[u] = a->coarse.cptr[i + 1];
#pragma unroll
        for (int q = 0; q < J; ++q)
          if (q * kWave < n) av[u][q] = a->coarse.Ainv[(int64_t)i * n + min(lane + q * kWave, n - 1)];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + u * kTailWaves >= n) break;
        at[u] = (int)a->coarse.cidx[min(c0[u], c1[u] - 1)];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + u * kTailWaves >= n) break;
        acc[u] = T(0);
#pragma unroll
        for (int q = 0; q < J; ++q)
          if (q * kWave < n) acc[u] = fma(av[u][q], bj[q], acc[u]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) acc[u] += __shfl_xor(acc[u], o, kWave);
        if (c0[u] < c1[u]) x[at[u]] = acc[u];
        for (int c = c0[u] + kWave; c < c1[u]; c += kWave) x[(int)a->coarse.cidx[c]] = acc[u];
      }
    }
    __syncthreads();
  }
  // ascent: levels lc + 1 .. lc + nlev - 1
  for (int k = 1; k < nlev; ++k) {
    F.load(a->lv[k]);
    F.prolong_from(a->lv[k - 1].N, vec(k - 1, 1), vec(k, 1));
    F.jacobi(vec(k, 1), vec(k, 2), vec(k, 0), post, omega, false);
  }
  if constexpr (LDS) {
    const V x = vec(nlev - 1, 1);
    T* g = a->lv[nlev - 1].x;
    for (int i = (int)threadIdx.x; i < (int)a->lv[nlev - 1].storage; i += kTailWG) g[i] = x[i];
  }
}

template <typename T, int DIM>
__global__ __launch_bounds__(kTailWG) void vcycle_tail_kernel(const Launch<TailArgs<T>> L) {
  const auto* a = resolve_ref(L, (int)blockIdx.x);
  if (a->lds > 0) tail_cycle<T, DIM, true>(a);
  else tail_cycle<T, DIM, false>(a);
}

template <typename T>
void run_tail(int dim, const Launch<TailArgs<T>>& l, int lds, hipStream_t s) {
  if (dim == 2) hipLaunchKernelGGL((vcycle_tail_kernel<T, 2>), dim3(l.nwg), dim3(kTailWG), lds, s, l);
  else hipLaunchKernelGGL((vcycle_tail_kernel<T, 3>), dim3(l.nwg), dim3(kTailWG), lds, s, l);
}

}  // namespace

template <typename T>
TailArgs<T> tail_args(const mf_mesh* m, int lc, int nlev, int pre, int post, double omega,
                      const std::vector<void*>& b, const std::vector<void*>& x, const std::vector<void*>& t) {
  TailArgs<T> a{};
  a.nlev = nlev;
  a.pre = pre;
  a.post = post;
  a.omega = (T)omega;
  a.coarse = coarse_args<T>(m->levels[lc], b[lc], x[lc]);
  for (int k = 0; k < nlev; ++k) a.lv[k] = tail_level<T>(m->levels[lc + k], b[lc + k], x[lc + k], t[lc + k]);
  int64_t lds = 0;
  for (int k = 0; k < nlev; ++k) lds += 3 * tail_lds_vec(a.lv[k].storage, (int)sizeof(T));
  a.lds = lds <= kTailLdsMax ? (int)lds : 0;
  return a;
}
template TailArgs<double> tail_args<double>(const mf_mesh*, int, int, int, int, double, const std::vector<void*>&,
                                            const std::vector<void*>&, const std::vector<void*>&);
template TailArgs<float> tail_args<float>(const mf_mesh*, int, int, int, int, double, const std::vector<void*>&,
                                          const std::vector<void*>&, const std::vector<void*>&);

int launch_vcycle_tail(const mf_mesh* m, int lc, int nlev, int dtype, int pre, int post, double omega,
                       const std::vector<void*>& b, const std::vector<void*>& x, const std::vector<void*>& t,
                       hipStream_t s) {
  if (nlev < 1 || nlev > kTailLevels) return set_error(MF_EINVAL, "tail levels out of range");
  if (dtype == MF_F64) {
    const TailArgs<double> a = tail_args<double>(m, lc, nlev, pre, post, omega, b, x, t);
    run_tail<double>(m->dim, single(a, 1), a.lds, s);
  } else {
    const TailArgs<float> a = tail_args<float>(m, lc, nlev, pre, post, omega, b, x, t);
    run_tail<float>(m->dim, single(a, 1), a.lds, s);
  }
  return check_launch();
}

int launch_tail_batch(const BatchOp& op, const char* table, hipStream_t s) {
  if (op.nwg <= 0) return MF_OK;
  // op.variant: the largest LDS size of the members (each member's own record says whether it uses LDS)
  if (op.dtype == MF_F64) run_tail<double>(op.dim, batched<TailArgs<double>>(op, table), op.variant, s);
  else run_tail<float>(op.dim, batched<TailArgs<float>>(op, table), op.variant, s);
  return check_launch();
}

}  // namespace mf

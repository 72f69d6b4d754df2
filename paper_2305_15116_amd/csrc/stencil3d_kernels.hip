// 3D constant-stencil kernels (gfx950): one launch finishes every row of a
// level (apply, weighted Jacobi, residual and norms).  Its tile list holds the
// interior walk's columns, the macro faces and the macro edge and vertex
// copies (walk3d.hpp), spread among each other.

#include <hip/hip_runtime.h>

#include <string>

#include "launch.hpp"
#include "walk3d.hpp"

namespace mf {

namespace {

template <typename T, int MODE, int R>
__global__ __launch_bounds__(kWG) void stencil3_kernel(const Launch<StencilArgs<T>> L) {
  const int g = R == kMaxR3 ? wave::xcd_wg_runs(L.nwg, wave::kRuns3) : wave::xcd_wg(L.nwg);
  if (g < 0) return;
  StencilArgs<T> a;
  const int n = resolve(L, g, a);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Tile t = load_seg(a.tiles, n * kWavesPerWG + wv);
  double ss = 0.0, mx = 0.0;
  if (t.macro >= 0) walk3<T, MODE, R>(t, a.md[t.macro], a.X, a.Y, a.B, a.omega, ss, mx);
  else if (t.macro == kFaceTile) face_rows<T, MODE>(a, t, ss, mx);
  else if (t.macro != -1) edge_rows<T, 3, MODE>(a, t, ss, mx);
  if (has_partials(MODE) && a.part != nullptr) wg_partial<kWavesPerWG>(ss, mx, a.part, a.np, n);
}

// Workgroups per CU of the fine levels' launches.  Cube at N = 256 / 512, us
// without a cap, then with 4 / 3 / 2: FP64 apply 72.9 / 507, 71.3 / 497, 70.6 /
// 474, 72.8 / 472; FP64 Jacobi 96.8 / 706, -, 94.5 / 682, 92.8 / 643; FP32 apply
// 41.0 / 274, 38.9 / 248, 39.7 / 255, -; FP32 Jacobi 47.8 / 374, 46.2 / 347, 46.8
// / 340, 51.3 / 367.
template <typename T, int MODE>
constexpr int wgs_per_cu() {
  return sizeof(T) == 4 ? 4 : (MODE == kApply ? 3 : 2);
}

template <typename T, int MODE>
int run(int R, const Launch<StencilArgs<T>>& l, hipStream_t s) {
  const dim3 grid(R == kMaxR3 ? wave::xcd_grid_runs(l.nwg, wave::kRuns3) : wave::xcd_grid(l.nwg)), wg(kWG);
  const int lds = R == kMaxR3 ? wave::lds_cap(l.nwg, wave::kRuns3.from, wgs_per_cu<T, MODE>(), partials_lds(MODE)) : 0;
  static_assert(kMaxR3 == 4, "one instance per band height");
  if (R == 4) hipLaunchKernelGGL((stencil3_kernel<T, MODE, 4>), grid, wg, lds, s, l);
  else if (R == 3) hipLaunchKernelGGL((stencil3_kernel<T, MODE, 3>), grid, wg, lds, s, l);
  else if (R == 2) hipLaunchKernelGGL((stencil3_kernel<T, MODE, 2>), grid, wg, lds, s, l);
  else if (R == 1) hipLaunchKernelGGL((stencil3_kernel<T, MODE, 1>), grid, wg, lds, s, l);
  else return set_error(MF_EINVAL, "internal: no 3D walk over bands of " + std::to_string(R) + " rows");
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? MF_OK : set_error(MF_EDEVICE, hipGetErrorString(e));
}

template <typename T>
int dispatch(int mode, int R, const Launch<StencilArgs<T>>& l, hipStream_t s) {
  if (l.nwg <= 0) return MF_OK;
  switch (mode) {
    case kApply: return run<T, kApply>(R, l, s);
    case kJacobi: return run<T, kJacobi>(R, l, s);
    case kJacobi2: return run<T, kJacobi2>(R, l, s);
    case kResidual: return run<T, kResidual>(R, l, s);
    case kNormB: return run<T, kNormB>(R, l, s);
    default: return run<T, kApplyDot>(R, l, s);
  }
}

}  // namespace

int launch_stencil3(int mode, int R, const Launch<StencilArgs<double>>& l, hipStream_t s) {
  return dispatch(mode, R, l, s);
}
int launch_stencil3(int mode, int R, const Launch<StencilArgs<float>>& l, hipStream_t s) {
  return dispatch(mode, R, l, s);
}

}  // namespace mf

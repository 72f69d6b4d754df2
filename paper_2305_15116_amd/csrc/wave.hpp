// Wavefront helpers shared by the stencil walks (device code, gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include "mf_internal.hpp"
#include "xcd.hpp"

namespace mf {
namespace wave {

// Cross-lane neighbours through DPP wavefront shifts (a VALU op, no LDS
// traffic): wave_shr:1 gives each lane the value of lane - 1, wave_shl:1 that
// of lane + 1.  Lanes 0 and 63, which have no source, receive 0 (bound_ctrl);
// they are halo lanes whose results are never stored.  Without an `old`
// operand the move needs no register copy of its source.
constexpr int kDppWaveShl1 = 0x130;
constexpr int kDppWaveShr1 = 0x138;

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  const int i = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(i, CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long l = __builtin_bit_cast(long long, v);
  const int lo = (int)(l & 0xffffffffLL), hi = (int)(l >> 32);
  const int rlo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, true);
  const int rhi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((long long)rhi << 32) | (long long)(unsigned)rlo);
}
template <typename T>
__device__ __forceinline__ T up1(T v) { return dpp_move<kDppWaveShr1>(v); }  // value of lane - 1
template <typename T>
__device__ __forceinline__ T dn1(T v) { return dpp_move<kDppWaveShl1>(v); }  // value of lane + 1

// This block's natural workgroup under the mappings of xcd.hpp.
__device__ __forceinline__ int xcd_wg(int nwg) { return xcd_wg_at(blockIdx.x, nwg); }
__device__ __forceinline__ int xcd_wg_runs(int nwg, XcdRuns r) { return xcd_wg_at(blockIdx.x, nwg, r); }
__device__ __forceinline__ int xcd_wg_lead(int nwg, int lead, int lead2, XcdRuns r) {
  return xcd_wg_at(blockIdx.x, nwg, lead, lead2, r);
}

// The 2D walks: runs of 32.  Level 14, FP64 apply / Jacobi: 380.7 / 565.6 us
// with runs of 32, 399 / 586 with one chunk per XCD, 384.8 / 566 and 377 / 564
// with 16 and 64 (two triangles at level 12: 58.0 / 82.3, 62.1 / 86.9, 58.3 /
// 82.2, 57.8 / 82.5); variable coefficient at level 14 604 -> 578, P2 at level 13
// 424 -> 415.  13 triangles at level 10: FP64 (3,600 workgroups) 31.6 -> 31.1,
// FP32 (1,900) 19.4 -> 20.4, one triangle at level 10 5.5 -> 5.7.
constexpr XcdRuns kRuns2{3000, 5};
// From this side on the 2D launches that gain from it cap their workgroups per CU
// (64 triangles at level 9, FP64 variable coefficient: 41.0 -> 39.0 us).  On shorter
// rows most tiles lie on a macro's boundary, whose latency needs the waves: variable
// coefficient, FP32, 3,200 triangles at levels 6 and 7 39.5 and 103 us without, 43.5
// and 116 with the cap (FP64 level 6 51.5 and 54.5); two FP32 sweeps at level 7 225 and
// 251.
constexpr int kCapN = 512;
// The 3D walks of fine levels: runs of 16.  N = 256, FP64 apply / Jacobi /
// residual 73.6 / 94.0 / 93.2 us against 75.3 / 96 / 96 with one chunk per XCD
// (runs of 4: 74.8 / 94.3 / 93.7, of 64: 76.8 / 98.9 / 98.7).
constexpr XcdRuns kRuns3{1000, 4};

}  // namespace wave
}  // namespace mf

// Internal types of the matrix-free P1 stencil library, shared by the host
// set-up code and the HIP kernels (never by the oracle).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#define MF_HD __host__ __device__ __forceinline__

namespace mf {

// ---------------------------------------------------------------- tiling
// One wavefront (64 lanes) owns 64 consecutive columns of a macro row and
// produces the 62 inner ones (lanes 0 and 63 are the halo); it walks a strip
// of rows upward, keeping the three rows the 2D stencil reads in registers
// (the layout of the paper's generated kernel: x fastest, rows bottom-up,
// Performance Modeling, experiment description).  Four waves form a workgroup.
constexpr int kWave = 64;
constexpr int kTileW = 62;
// Short strips keep the rows written at any moment within a few MB, so the
// partial cache lines at wave boundaries are completed in L2 before write-back.
#ifndef MF_TILE_H2
#define MF_TILE_H2 8
#endif
constexpr int kTileH2 = MF_TILE_H2;   // rows per 2D wave tile (FP64)
// FP32 rows carry half the bytes: taller tiles with a deeper load ring keep
// as many bytes in flight per wave.
constexpr int kTileH2F = 16;
// A launch whose workgroups all run at once takes as long as one tile: levels
// take the lowest tiles of which they need at most kShortWGs workgroups (four
// per CU), FP32 levels of at most kMidWGs of kTileH2 rows take those.  FP64 and
// FP32 Jacobi, us, against kTileH2 and kTileH2F rows: one triangle at level 8 5.3 ->
// 3.3 and 7.3 -> 3.0, seven at level 7 5.8 -> 3.7 and 7.5 -> 3.4 (2 rows), seven at level
// 8 5.9 -> 5.0 and 7.6 -> 4.1 (4 rows), 22 at level 8 FP32 9.4 -> 7.2.
constexpr int kTileShort[2] = {2, 4};
constexpr int kShortWGs = 1024, kMidWGs = 1024;
// 3D: a wave takes 64 consecutive columns of a slab of PZ slices, cut into
// bands of R rows, and walks them upward through the slices (walk3d.hpp).
// Measured on the 6-tet cube (us per launch, FP64 apply / Jacobi / residual):
// large bands read fewer rows twice and win where memory bounds the launch
// (N = 256: R = 4 74 / 96 / 96, R = 2 86 / 102 / 101), short slabs keep the
// launch's front compact (PZ = 4 / 6 / 8: 73 / 75 / 75; 8 from N = 512 on, for
// fewer norm partials); small levels need waves instead (N = 128: R = 3
// 11.7 / 12.9 / 12.8, R = 4 12.6 / 15.8 / 15.6; N = 64: R = 2 4.9 / 5.5 / 5.3, R = 1
// 5.5 / 6.0 / 5.7; N = 32: R = 1 4.4 / 5.0 / 4.5, R = 2 4.5 / 5.1 / 5.0).
struct Shape3 {
  int R, PZ;  // rows per band, slices per slab
};
MF_HD constexpr Shape3 shape3(int N) {
  return N >= 512 ? Shape3{4, 8} : N >= 256 ? Shape3{4, 6} : N >= 128 ? Shape3{3, 4} : N >= 64 ? Shape3{2, 4} : Shape3{1, 2};
}
constexpr int kMaxR3 = 4;
// The variable-coefficient walk's: it forms R + 1 rows and PZ + 1 layers of
// cells for the R x PZ points of a column, and holds the rows of two vectors
// (FP64 R = 3 spills).  Cube, us per apply with the boundary in a launch of its own
// (in the walk's launch the shapes taken are at 126, 62 and 21): N = 256 FP64 R = 2, PZ = 8
// / 12 / 6 145 / 143 / 154, R = 1 159; FP32 R = 3, PZ = 12 / 8 77.0 / 78.5, R = 4, PZ = 8
// 81.3, R = 2 79.5; N = 128 FP64 R = 2 29.8, R = 3 47.
MF_HD constexpr Shape3 shape3_varcoef(int N, bool f32) {
  return N >= 256 ? (f32 ? Shape3{3, 12} : Shape3{2, 12}) : N >= 64 ? Shape3{2, 4} : Shape3{1, 2};
}
// Kinds of a 3D tile list's other tiles (Tile::macro): inner points of a macro
// face, copies of macro edge and vertex DoFs.
constexpr int kFaceTile = -2;
constexpr int kEdgeTile = -3;
constexpr int kEdgeBigTile = -4;
// From this side on the inner points of a face have tiles of their own; below
// (at most 21 points) they are listed with the edge and vertex copies.
constexpr int kMinFaceN = 16;
// Points per face tile: Dirichlet faces (copies), faces of one and of two
// macros.  Up to N = 128 a launch is a few latencies long, and a tile that takes
// a second step lengthens it (N = 32, FP64 apply 4.5 us with 64 points, 6.6
// with 128); above, larger tiles keep the norm partials few.
struct FaceRuns {
  int dirichlet, one, two;
};
constexpr FaceRuns kFaceRunsWG{1024, 256, 128};  // where a workgroup takes a tile
MF_HD constexpr FaceRuns face_runs(int N) { return N >= 256 ? FaceRuns{2048, 1536, 128} : FaceRuns{256, 64, 64}; }
#ifndef MF_WAVES_PER_WG
#define MF_WAVES_PER_WG 4
#endif
constexpr int kWavesPerWG = MF_WAVES_PER_WG;
constexpr int kWG = kWave * kWavesPerWG;
constexpr int kIfaceWG = 256;  // groups per interface workgroup
constexpr int kXCD = 8;        // MI355X: 8 accelerator complex dies, workgroups dealt round-robin

// A wave tile: columns [x0, x0+62) of rows [y0, y0+H) of `macro` (2D); the
// columns from x0 on of the slab's y0 at slices z & 0xffff on, z >> 16 of them (3D); y0 points of face z from point x0 on (kFaceTile);
// y0 copies from copy x0 on (kEdgeTile, kEdgeBigTile).  For per-point kernels the same record names a row
// segment of 64 points starting at x0 of row y0 in slice z.  macro = -1: padding.
struct Tile {
  int32_t macro, x0, y0, z;
};

// A copy of a macro-boundary DoF: macro id and its index-space point.
struct Copy {
  int32_t macro, x, y, z;
};

// A macro face (3D): the one or two macros that contain it.  An inner point has
// face weights wa, wb >= 1 and wc = N - wa - wb >= 1; in macro cp[i] it is the
// point n N + a wa + b wb (per coordinate).
struct FaceCopy {
  int32_t macro;
  int8_t face;  // the macro's face: 0: x + y + z = N, 1..3: x, y, z = 0
  int8_t n[3], a[3], b[3];
};
struct FaceDev {
  int32_t N;
  int16_t copies, dirichlet;
  FaceCopy cp[2];  // (one macro: repeated)
  double inv;      // 1 / assembled diagonal of an inner point
  float invf;
};

// A copy of a macro edge or vertex DoF (2D: of a shared one; 3D below kMinFaceN: of
// a face point too).
struct EdgeCopy {
  int64_t idx;  // storage index
  int32_t macro;
  uint16_t x, y, z;
  uint8_t mask;          // support mask in its macro
  uint8_t head, copies;  // lane of the DoF's first copy in its tile, number of copies (kEdgeTile)
  uint8_t dirichlet;
  EdgeCopy() {}  // (left unset: lists of them are filled by several threads)
};

// Per-macro, per-level constants.  wm[s] is the (partial) stencil of a point
// whose non-zero barycentric weights are the local vertices in mask s: the
// sum, over the micro-elements of this macro containing the point, of its
// rows of the element matrices.  s = full (7 in 2D, 15 in 3D) is the
// interior stencil; faces, edges and vertices of the macro get the rows of
// the elements on their side only, which copies of a shared DoF then sum.
// Element matrices K[t] are stored as 4x4 (2D uses the leading 3x3).
struct MacroDev {
  int64_t base;         // storage offset of the macro
  int64_t vid[4];       // global vertex ids in cell order (for keys)
  int32_t N;
  uint16_t own_mask;    // bit s: this macro owns the primitive spanned by local-vertex subset s
  uint16_t dir_mask;    // bit s: that primitive lies on the Dirichlet boundary
  uint16_t shared_mask; // bit s: that primitive belongs to more than one macro
  uint16_t pad0_;
  float inv_diagf;
  double inv_diag;      // 1 / interior centre weight
  double wm[16][16];
  float wmf[16][16];
  double K[6][16];      // element matrix of each micro-element type (row-major 4 x 4)
  float Kf[6][16];      // the same in FP32 (FP32 kernels read it without conversions)
  double zinv[16];      // 1 / assembled diagonal of the points with support s, 0 on the Dirichlet boundary
  float zinvf[16];
};

// ---------------------------------------------------------------- layout
MF_HD int64_t tet_count(int64_t n) { return n * (n + 1) * (n + 2) / 6; }
MF_HD int64_t tri_count(int64_t n) { return n * (n + 1) / 2; }
// storage points of one macro
MF_HD int64_t macro_points(int dim, int64_t N) { return dim == 2 ? tri_count(N + 1) : tet_count(N + 1); }
// Tet(n) for 0 <= n < 2^16 with 32-bit divisions by constants only (device
// index math runs on the scalar unit, where 64-bit division is a long
// sequence): n(n+1)/2 is an integer, and one of n, n+1, n+2 is a multiple of 3.
MF_HD int64_t tet_count_small(int n) {
  const uint32_t t = (uint32_t)n * (uint32_t)(n + 1) / 2u;
  return (n % 3 == 1) ? (int64_t)t * (int64_t)((n + 2) / 3) : (int64_t)(t / 3u) * (int64_t)(n + 2);
}
// first index of slice z (3D, N <= 2048)
MF_HD int64_t slice_base(int N, int z) { return tet_count_small(N + 1) - tet_count_small(N + 1 - z); }
// start of row y in a triangle of side M (M < 2^15: fits 32 bits)
MF_HD int32_t row_start(int M, int y) { return y * (M + 2) - ((y * (y + 1)) >> 1); }
MF_HD int64_t idx2(int N, int x, int y) { return (int64_t)row_start(N, y) + x; }
MF_HD int64_t idx3(int N, int x, int y, int z) { return slice_base(N, z) + row_start(N - z, y) + x; }

// ---------------------------------------------------------------- micro-elements
// Index-space vertex offsets of the micro-element types (Bey's refinement in
// the lattice; 2D: the up and down triangles).  An element of type t with
// anchor a exists iff a >= 0 componentwise and sum(a) <= N - slack[t].
struct ElemTable {
  int ntypes;
  int nv;
  int8_t off[6][4][3];
  int8_t slack[6];
};

MF_HD constexpr ElemTable elem_table(int dim) {
  if (dim == 2)
    return ElemTable{2, 3,
                     {{{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 0}},
                      {{1, 0, 0}, {1, 1, 0}, {0, 1, 0}, {0, 0, 0}},
                      {}, {}, {}, {}},
                     {1, 2, 0, 0, 0, 0}};
  // 3D: up tet; the octahedron around the (0,1,0)-(1,0,1) diagonal with ring
  // (1,0,0),(1,1,0),(0,1,1),(0,0,1); down tet.
  return ElemTable{6, 4,
                   {{{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}},
                    {{0, 1, 0}, {1, 0, 1}, {1, 0, 0}, {1, 1, 0}},
                    {{0, 1, 0}, {1, 0, 1}, {1, 1, 0}, {0, 1, 1}},
                    {{0, 1, 0}, {1, 0, 1}, {0, 1, 1}, {0, 0, 1}},
                    {{0, 1, 0}, {1, 0, 1}, {0, 0, 1}, {1, 0, 0}},
                    {{1, 1, 0}, {1, 0, 1}, {0, 1, 1}, {1, 1, 1}}},
                   {1, 2, 2, 2, 2, 3}};
}

// Stencil offsets in weight order (see mf_stencil.h).
struct StencilTable {
  int n;
  int centre;
  int8_t off[15][3];
};

MF_HD constexpr StencilTable stencil_table(int dim) {
  if (dim == 2)
    return StencilTable{7, 3, {{0, -1, 0}, {1, -1, 0}, {-1, 0, 0}, {0, 0, 0}, {1, 0, 0}, {-1, 1, 0}, {0, 1, 0}}};
  return StencilTable{15, 7,
                      {{0, 0, -1}, {1, 0, -1}, {0, 1, -1}, {-1, 1, -1},
                       {0, -1, 0}, {1, -1, 0}, {-1, 0, 0}, {0, 0, 0}, {1, 0, 0}, {-1, 1, 0}, {0, 1, 0},
                       {0, -1, 1}, {1, -1, 1}, {-1, 0, 1}, {0, 0, 1}}};
}

MF_HD constexpr int full_mask(int dim) { return dim == 2 ? 7 : 15; }

// Local-vertex support mask of point p of a macro: bit k set iff barycentric
// weight k is non-zero (weights (N - sum p, p1, .., pd)).
MF_HD int support_mask(int dim, int N, int x, int y, int z) {
  const int w0 = N - x - y - (dim == 3 ? z : 0);
  int m = (w0 != 0 ? 1 : 0) | (x != 0 ? 2 : 0) | (y != 0 ? 4 : 0);
  if (dim == 3) m |= (z != 0 ? 8 : 0);
  return m;
}

// Operation modes of the fused stencil kernels.
enum Mode : int {
  kApply = 0,     // y = A x
  kJacobi = 1,    // y = x + omega D^-1 (b - A x)
  kResidual = 2,  // y = b - A x  (+ sum of squares and max |.| partials)
  kNormB = 3,     // no output; partials of b only (||b|| over unique DoFs)
  kApplyDot = 4,  // y = A x  (+ partials of x . y over unique DoFs)
  kJacobi2 = 5,   // two Jacobi sweeps from a zero iterate, y = z + omega D^-1 (b - A z) with z = omega D^-1 b
};

// Modes whose kernels leave (sum, max) partials.
MF_HD constexpr bool has_partials(int mode) { return mode == kResidual || mode == kNormB || mode == kApplyDot; }

// Interface-kernel-only modes.
enum IfaceMode : int {
  kDirichletSet = 11,  // y = b at Dirichlet DoFs only
};

}  // namespace mf

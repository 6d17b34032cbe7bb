// Device helpers shared by the multigrid kernels of the single-request
// (mg_kernels.hip) and batched (mg_batch.hip) W-cycles: vector loads, the
// Q1 prolongation coefficients and the geometry of the RAS blocks (Section
// 4.2: a 4 x 4 core of squares plus the layer of squares across its faces).
//
// Block slots p < 32 of a tile: 0..15 the core (x = p % 4, y = p / 4), then
// the layer x = -1, x = 4, y = -1, y = 4 (4 squares each).  Extended slots
// 32..51 add the squares at distance 1 outside the block: x = -2, x = 5,
// y = -2, y = 5 (4 each) and the 4 diagonal corners.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dcg {
namespace mg {

// Four consecutive values of the library's own buffers (16-byte aligned).
__device__ __forceinline__ void ld4(const float* p, float v[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void ld4(const double* p, double v[4]) {
  const double2 a = reinterpret_cast<const double2*>(p)[0];
  const double2 b = reinterpret_cast<const double2*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ __forceinline__ void st4(float* p, const float v[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void st4(double* p, const double v[4]) {
  reinterpret_cast<double2*>(p)[0] = make_double2(v[0], v[1]);
  reinterpret_cast<double2*>(p)[1] = make_double2(v[2], v[3]);
}

// The same for the vectors of a caller, which are aligned to their elements only (a
// slice may start anywhere): gfx950 makes a 16-byte global access at any 4-byte
// address, and the compiler emits the same instructions as for aligned vectors.
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef double double2_any __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ double2 ld2_any(const double* p) {
  const double2_any t = *reinterpret_cast<const double2_any*>(p);
  return make_double2(t.x, t.y);
}
__device__ __forceinline__ void st2_any(double* p, double x, double y) {
  *reinterpret_cast<double2_any*>(p) = double2_any{x, y};
}
__device__ __forceinline__ void ld4_any(const float* p, float v[4]) {
  const float4_any t = *reinterpret_cast<const float4_any*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void ld4_any(const double* p, double v[4]) {
  const double2 a = ld2_any(p), b = ld2_any(p + 2);
  v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ __forceinline__ void st4_any(float* p, const float v[4]) {
  *reinterpret_cast<float4_any*>(p) = float4_any{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ void st4_any(double* p, const double v[4]) {
  st2_any(p, v[0], v[1]);
  st2_any(p + 2, v[2], v[3]);
}

// 16 x 16 x 4 MFMA of the level type.  Operand lanes: A holds (row l % 16,
// k l / 16), B holds (k l / 16, column l % 16).  The accumulator of lane l
// holds column l % 16 and rows 4 (l / 16) + v (FP32) or 4 v + l / 16 (FP64),
// v = 0..3.
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mac(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mac(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// Coefficient of coarse corner A at fine corner a of child ch (exact).
template <typename T>
__device__ __forceinline__ T pcoef(int ch, int a, int A) {
  const int px = (ch & 1) + (a & 1), py = (ch >> 1) + (a >> 1);
  const int wx = (A & 1) ? px : 2 - px, wy = (A >> 1) ? py : 2 - py;
  return T(wx * wy) * T(0.25);
}

// acc += the four rows of a square's operator blocks times the five squares of its
// stencil, the blocks of class ``cls`` of a table [9][5][4][4] through scalar loads:
// one pass per class present in the wavefront, interior wavefronts hold one.
template <typename T>
__device__ __forceinline__ void class_rows(const T* __restrict__ Lc, int cls, const T (&zq)[5][4],
                                           T (&acc)[4]) {
  for (;;) {
    const int c = __builtin_amdgcn_readfirstlane(cls);
    if (cls != c) continue;
    const T* l = Lc + 80 * c;
#pragma unroll
    for (int s = 0; s < 5; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[j] += l[16 * s + 4 * j] * zq[s][0] + l[16 * s + 4 * j + 1] * zq[s][1] +
                  l[16 * s + 4 * j + 2] * zq[s][2] + l[16 * s + 4 * j + 3] * zq[s][3];
    break;
  }
}

// Pending slot (3 e + rank) of tile t's output at square (X, Y) of its block, and the
// weight of the average.  Blocks containing (X, Y): its core tile T and the
// neighbour tile on each side where the square lies on T's core edge; the slot is
// this tile's rank among them in increasing order.
template <typename T>
__device__ __forceinline__ int64_t pending_slot(int X, int Y, int n, int t, T& w) {
  const int tpr = n >> 2, TX = X >> 2, TY = Y >> 2, lx = X & 3, ly = Y & 3, Tc = TY * tpr + TX;
  const bool below = ly == 0 && TY > 0, left = lx == 0 && TX > 0;
  const bool right = lx == 3 && TX < tpr - 1, above = ly == 3 && TY < tpr - 1;
  const int count = 1 + below + left + right + above;
  const int rank = (below && Tc - tpr < t) + (left && Tc - 1 < t) + (Tc < t) +
                   (right && Tc + 1 < t) + (above && Tc + tpr < t);
  w = count == 1 ? T(1) : (count == 2 ? T(0.5) : T(1.0 / 3.0));
  return 3 * ((int64_t)Y * n + X) + rank;
}

// Position (relative to the tile origin) of block slot p < 32.
__device__ __forceinline__ void slot_pos(int p, int& px, int& py) {
  if (p < 16) { px = p & 3; py = p >> 2; }
  else if (p < 20) { px = -1; py = p - 16; }
  else if (p < 24) { px = 4; py = p - 20; }
  else if (p < 28) { px = p - 24; py = -1; }
  else { px = p - 28; py = 4; }
}

// Extended slot (0..51) of the position, -1 outside the pattern.
__device__ __forceinline__ int pos_slot(int px, int py) {
  const bool cx = px >= 0 && px < 4, cy = py >= 0 && py < 4;
  if (cx && cy) return py * 4 + px;
  if (cy) {
    if (px == -1) return 16 + py;
    if (px == 4) return 20 + py;
    if (px == -2) return 32 + py;
    if (px == 5) return 36 + py;
    return -1;
  }
  if (cx) {
    if (py == -1) return 24 + px;
    if (py == 4) return 28 + px;
    if (py == -2) return 40 + px;
    if (py == 5) return 44 + px;
    return -1;
  }
  if (px == -1 && py == -1) return 48;
  if (px == 4 && py == -1) return 49;
  if (px == -1 && py == 4) return 50;
  if (px == 4 && py == 4) return 51;
  return -1;
}

__device__ __forceinline__ int nbr_slot(int p, int s) {
  int px, py;
  slot_pos(p, px, py);
  const int dx = s == 1 ? -1 : (s == 2 ? 1 : 0);
  const int dy = s == 3 ? -1 : (s == 4 ? 1 : 0);
  return pos_slot(px + dx, py + dy);
}

// Position (relative to the tile origin) of extended slot q < 52.
__device__ __forceinline__ void ext_pos(int q, int& px, int& py) {
  if (q < 32) { slot_pos(q, px, py); return; }
  if (q < 36) { px = -2; py = q - 32; }
  else if (q < 40) { px = 5; py = q - 36; }
  else if (q < 44) { px = q - 40; py = -2; }
  else if (q < 48) { px = q - 44; py = 5; }
  else { px = (q & 1) ? 4 : -1; py = (q < 50) ? -1 : 4; }
}

// Square of extended slot q of tile t on an n x n grid (-1 outside).
__device__ __forceinline__ int ext_square(int t, int q, int n) {
  const int tpr = n >> 2;
  int px, py;
  ext_pos(q, px, py);
  const int x = 4 * (t % tpr) + px, y = 4 * (t / tpr) + py;
  return (x < 0 || y < 0 || x >= n || y >= n) ? -1 : y * n + x;
}

// Workgroups are dispatched to the 8 XCDs (each with its own L2) round-robin
// by workgroup id.  Tiles that share squares (the layer and the outside
// neighbours of a block) should be handled by the same XCD, so workgroup b
// takes logical index (b mod 8) * (G / 8) + b / 8: XCD x processes the
// contiguous range x G / 8 .. (x + 1) G / 8 - 1 (a band of tile rows).  Only
// grids of at most kXcdBandMaxGrid workgroups are remapped: the largest
// grids stream their factors from HBM, where the eight separate fronts of
// the band order measured slower (4 % at n = 512) while the cache-resident
// levels gain 5-20 %.  Grids not divisible by 8 keep the identity.
#ifndef DCG_XCD_BAND_MAX_GRID
#define DCG_XCD_BAND_MAX_GRID 2048
#endif
constexpr int kXcdBandMaxGrid = DCG_XCD_BAND_MAX_GRID;
__device__ __forceinline__ int xcd_band_index(int b, int G) {
  return ((G & 7) || G > kXcdBandMaxGrid) ? b : (b & 7) * (G >> 3) + (b >> 3);
}

// The same order without the size limit, for launches that stream vectors only
// (each XCD then reads contiguous rows of squares).
__device__ __forceinline__ int xcd_band(int b, int G) {
  return (G & 7) ? b : (b & 7) * (G >> 3) + (b >> 3);
}

// Class of the tile (TX, TY), tpr tiles per side, from the packed classes of the
// nine tile positions (first / inner / last along each axis, 4 bits each at
// 3 cy + cx).
__host__ __device__ __forceinline__ int tile_class_of(uint64_t cls9, int TX, int TY, int tpr) {
  const int cx = TX == 0 ? 0 : (TX == tpr - 1 ? 2 : 1), cy = TY == 0 ? 0 : (TY == tpr - 1 ? 2 : 1);
  return int(cls9 >> (4 * (3 * cy + cx))) & 15;
}

// Index of block (P, Q), P <= Q, in the packed upper-triangular order
// (row by row) of the symmetric tile inverses.
__host__ __device__ constexpr int blk_index(int P, int Q) { return P * (15 - P) / 2 + Q; }

}  // namespace mg
}  // namespace dcg

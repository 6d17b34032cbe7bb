// Batched W-cycle kernels: the multigrid steps of mg_kernels.hip (Algorithm 4
// with the RAS smoother of Section 4.2) applied to kBatch requests that share
// one mesh.  Level vectors are request-interleaved, [square][request][4], so
// that a square's values of all requests are one contiguous 256 B (FP32) or
// 512 B (FP64) run.
//
// The RAS step is where batching changes the arithmetic shape: for one
// request the tile solve u = (L_k)_t^{-1} r is a 128 x 128 matrix-vector
// product bound by the factor stream; for kBatch requests it is a
// 128 x 128 by 128 x kBatch product, done with v_mfma_*_16x16x4 (FP32 or
// FP64 by the level type) so that the factor bytes are paid once for all
// requests.  Column c of every MFMA output reads column c of the operand
// only, so a request's result does not depend on which other requests share
// the batch.
#include <type_traits>

#include "kernels.hpp"
#include "mg_common.hpp"

namespace dcg {
namespace {
using namespace mg;

constexpr int kThreads = 256;
constexpr int B = kBatch;
constexpr int kCoarse = 1024;   // dofs of the 16 x 16 coarsest level

__device__ __forceinline__ int64_t at(int64_t e, int c) { return (e * B + c) * 4; }

// z += pending tile outputs of square e, request c (blocks in increasing
// order; unused cover slots hold zeros).
template <typename T>
__device__ __forceinline__ void add_pending_b(const T* Ye, int64_t e, int c, T z[4]) {
  T y0[4], y1[4], y2[4];
  ld4(Ye + at(3 * e, c), y0);
  ld4(Ye + at(3 * e + 1, c), y1);
  ld4(Ye + at(3 * e + 2, c), y2);
#pragma unroll
  for (int j = 0; j < 4; ++j) z[j] = ((z[j] + y0[j]) + y1[j]) + y2[j];
}

// Loads of square e, request c: z_old, pending Y, and with PROL the coarse z and its
// pending Y; z_new from them.
template <typename T, bool PROL>
__device__ __forceinline__ void load_z_b(const SweepArgs<T>& a, int e, int c, T (&v)[PROL ? 8 : 4][4]) {
#pragma unroll
  for (int i = 0; i < (PROL ? 8 : 4); ++i) v[i][0] = v[i][1] = v[i][2] = v[i][3] = T(0);
  if (e < 0) return;
  if (a.has_z) ld4(a.z_old + at(e, c), v[0]);
  if (a.has_y)
#pragma unroll
    for (int i = 0; i < 3; ++i) ld4(a.Y_old + at(3 * (int64_t)e + i, c), v[1 + i]);
  if constexpr (PROL) {
    const int E = ((e / a.n) >> 1) * a.nc + ((e % a.n) >> 1);
    ld4(a.zc + at(E, c), v[4]);
    if (a.c_has_y)
#pragma unroll
      for (int i = 0; i < 3; ++i) ld4(a.Yc + at(3 * (int64_t)E + i, c), v[5 + i]);
  }
}

template <typename T, bool PROL>
__device__ __forceinline__ void combine_z_b(const SweepArgs<T>& a, int e, const T (&v)[PROL ? 8 : 4][4],
                                            T (&z)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    z[j] = v[0][j];
    if (a.has_y) z[j] = ((z[j] + v[1][j]) + v[2][j]) + v[3][j];
  }
  if constexpr (PROL) {
    if (e < 0) return;
    const int ch = ((e % a.n) & 1) + 2 * ((e / a.n) & 1);
    T ec[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      ec[j] = v[4][j];
      if (a.c_has_y) ec[j] = ((ec[j] + v[5][j]) + v[6][j]) + v[7][j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      z[j] += pcoef<T>(ch, j, 0) * ec[0] + pcoef<T>(ch, j, 1) * ec[1] +
              pcoef<T>(ch, j, 2) * ec[2] + pcoef<T>(ch, j, 3) * ec[3];
  }
}

// One RAS step of level k for kBatch requests, NS workgroups of NW wavefronts per tile:
//   1. z on the 52 squares near the tile: z_old + pending Y [+ P e_coarse],
//      kept in LDS, the loads of two squares per thread in flight at a time; the
//      core squares are written to z_new;
//   2. U = f - L_k z on the 32 block squares (128 x kBatch), in LDS;
//   3. (L_k)_t^{-1} U in 16 x 16 row and column blocks x 4 MFMA k-steps; with
//      NS > 1 a workgroup computes a part of the row blocks, KS wavefronts share the
//      contraction of one;
//   4. Y_t = D_t U written to the pending slot of each block square.
//
// Small levels are a chain of latencies, so they run 8 wavefronts per tile, split
// over four workgroups where those fit the compute units at once: in FP64 n = 32
// 12.8 -> 9.8, n = 64 13.9 -> 11.9 us (FP32 9.3 -> 7.4).  n = 128 is bound by the bytes of
// the overlapping frames (3.25 z and pending sets per core square) and the MFMA rate,
// 37.6 -> 36.0 us; more workgroups in flight make it slower (35.4 and 44.4 us of a plain and
// a prolongating step at 3 per compute unit against 34.3 and 40.9 at 2).
template <typename T, bool PROL, int NW, int NS>
__global__ __launch_bounds__(64 * NW) void k_sweep_b(SweepArgs<T> a) {
  using V = typename Mfma<T>::v4;
  constexpr int NTH = 64 * NW, RB = 8 / NS;
  constexpr int HP = RB > NW ? RB / NW : 1;   // row blocks per wavefront
  constexpr int KS = NW > RB ? NW / RB : 1;   // wavefronts per row block
  constexpr int NQ = 8 / KS;                  // column blocks per wavefront
  constexpr int PD = NQ < 4 ? NQ : 4;         // of them requested ahead
  constexpr int NI = (52 * B + NTH - 1) / NTH, NF = 32 * B / NTH;
  constexpr int CH = 2;                       // squares in flight per thread
  __shared__ __align__(16) T zn[52][B][4];
  __shared__ __align__(16) T ul[32][B][4];
  const int part = NS > 1 ? blockIdx.x / a.tiles : 0;
  const int t = xcd_band_index(blockIdx.x - part * a.tiles, a.tiles);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, k = lane >> 4;
  int Pw[HP];
  Pw[0] = part * RB + wave % RB;
  if constexpr (HP == 2) Pw[1] = 7 - wave;
  const int Q0 = wave / RB * NQ;
  const bool need_z = a.has_z || a.has_y || PROL;

  T fr[NF][4];
#pragma unroll
  for (int u = 0; u < NF; ++u) {
    const int it = tid + u * NTH, e = ext_square(t, it / B, a.n);
    fr[u][0] = fr[u][1] = fr[u][2] = fr[u][3] = T(0);
    if (e >= 0) ld4(a.f + at(e, it % B), fr[u]);
  }
  if (need_z) {
#pragma unroll
    for (int u0 = 0; u0 < NI; u0 += CH) {
      T v[CH][PROL ? 8 : 4][4];
      int es[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int it = tid + (u0 + u) * NTH;
        es[u] = it < 52 * B ? ext_square(t, it / B, a.n) : -1;
        load_z_b<T, PROL>(a, es[u], it % B, v[u]);
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int it = tid + (u0 + u) * NTH;
        if (it >= 52 * B) continue;
        T z[4];
        combine_z_b<T, PROL>(a, es[u], v[u], z);
        st4(&zn[it / B][it % B][0], z);
        if (a.write_z && part == 0 && it < 16 * B) st4(a.z_new + at(es[u], it % B), z);
      }
    }
  }

  // MFMA A operands: lane (r, k) of k-step kk holds row 16 P + r, column
  // 16 Q + 4 k + kk of the tile inverse, one vector of the operand-order copy,
  // requested before the residual is formed
  const int tpr = a.n >> 2;
  const T* Ft = a.Fm + (int64_t)tile_class_of(a.cls9, t % tpr, t / tpr, tpr) * (64 * 256);
  auto load_q = [&](int Q, T (&dst)[HP][4]) {
#pragma unroll
    for (int h = 0; h < HP; ++h) ld4(Ft + ((Pw[h] * 8 + Q0 + Q) * 64 + lane) * 4, dst[h]);
  };
  T av[PD][HP][4];
#pragma unroll
  for (int Q = 0; Q < PD; ++Q) load_q(Q, av[Q]);
  __syncthreads();

  // U = f - L_k z: thread (block square p, request c), the four rows from the class
  // table in scalar registers (a wavefront holds four squares)
#pragma unroll
  for (int u = 0; u < NF; ++u) {
    const int it = tid + u * NTH, p = it / B, c = it % B;
    const int e = ext_square(t, p, a.n);
    if (e >= 0 && need_z) {
      T zq[5][4], acc[4] = {T(0), T(0), T(0), T(0)};
      const int ex = e % a.n, ey = e / a.n;
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int dx = s == 1 ? -1 : (s == 2 ? 1 : 0), dy = s == 3 ? -1 : (s == 4 ? 1 : 0);
        zq[s][0] = zq[s][1] = zq[s][2] = zq[s][3] = T(0);
        if (ex + dx >= 0 && ex + dx < a.n && ey + dy >= 0 && ey + dy < a.n)
          ld4(&zn[nbr_slot(p, s)][c][0], zq[s]);
      }
      class_rows(a.Lc, square_class(ex, ey, a.n), zq, acc);
#pragma unroll
      for (int j = 0; j < 4; ++j) fr[u][j] -= acc[j];
    }
    st4(&ul[p][c][0], fr[u]);
  }
  __syncthreads();

  // MFMA B operand of column block Q: lane (k, c = r) holds U[16 Q + 4 k + kk][c]
  V accs[HP];
#pragma unroll
  for (int h = 0; h < HP; ++h) accs[h] = V{T(0), T(0), T(0), T(0)};
#pragma unroll
  for (int Q = 0; Q < NQ; ++Q) {
    T bq[4], aq[HP][4];
    ld4(&ul[4 * (Q0 + Q) + k][r][0], bq);
#pragma unroll
    for (int h = 0; h < HP; ++h)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) aq[h][kk] = av[Q % PD][h][kk];
    if (Q + PD < NQ) load_q(Q + PD, av[Q % PD]);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int h = 0; h < HP; ++h) accs[h] = Mfma<T>::mac(aq[h][kk], bq[kk], accs[h]);
  }
  if constexpr (KS > 1) {          // the parts of a row block's contraction, in z's place
    T (*red)[4] = &zn[0][0];
    T out[4] = {accs[0][0], accs[0][1], accs[0][2], accs[0][3]};
    st4(red[tid], out);
    __syncthreads();
    if (wave >= RB) return;
#pragma unroll
    for (int p = 1; p < KS; ++p) {
      T o[4];
      ld4(red[tid + 64 * RB * p], o);
#pragma unroll
      for (int v = 0; v < 4; ++v) accs[0][v] += o[v];
    }
  }

  // FP32 lanes hold rows 4 k + v of row block P (square 4 P + k, corner v), FP64
  // lanes rows 4 v + k (square 4 P + v, corner k); request r
  constexpr int NO = std::is_same<T, float>::value ? 1 : 4;
#pragma unroll
  for (int h = 0; h < HP; ++h)
#pragma unroll
    for (int v = 0; v < NO; ++v) {
      const int e = ext_square(t, 4 * Pw[h] + (NO == 1 ? k : v), a.n);
      if (e < 0) continue;
      T w;
      const int64_t o = at(pending_slot(e % a.n, e / a.n, a.n, t, w), r);
      if constexpr (NO == 1) {
        const T y[4] = {w * accs[h][0], w * accs[h][1], w * accs[h][2], w * accs[h][3]};
        st4(a.Y_new + o, y);
      } else {
        a.Y_new[o + k] = w * accs[h][v];
      }
    }
}

// Pending update + residual + restriction for kBatch requests: one
// wavefront per coarse square, lane = (child, request); the four children's
// restricted contributions are summed across lanes.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_restrict_res_b(RestrictArgs<T> a) {
  const int nc = a.n >> 1;
  const int E = xcd_band_index(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6);
  if (E >= nc * nc) return;   // whole wavefronts
  const int ch = (threadIdx.x >> 4) & 3, c = threadIdx.x & 15;
  const int EX = E % nc, EY = E / nc;
  const int ex = 2 * EX + (ch & 1), ey = 2 * EY + (ch >> 1);
  const int e = ey * a.n + ex;
  T acc[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const int dx = s == 1 ? -1 : (s == 2 ? 1 : 0), dy = s == 3 ? -1 : (s == 4 ? 1 : 0);
    if (ex + dx < 0 || ex + dx >= a.n || ey + dy < 0 || ey + dy >= a.n) continue;
    const int cn = e + dy * a.n + dx;
    T z[4] = {T(0), T(0), T(0), T(0)};
    if (a.has_z) ld4(a.z_old + at(cn, c), z);
    if (a.has_y) add_pending_b(a.Y_old, cn, c, z);
    if (s == 0 && a.write_z) st4(a.z_new + at(e, c), z);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      T l[4];
      ld4(a.Lc + (square_class(ex, ey, a.n) * 5 + s) * 16 + 4 * j, l);
      acc[j] += l[0] * z[0] + l[1] * z[1] + l[2] * z[2] + l[3] * z[3];
    }
  }
  T rv[4];
  ld4(a.f + at(e, c), rv);
#pragma unroll
  for (int j = 0; j < 4; ++j) rv[j] -= acc[j];
  T ck[4];
#pragma unroll
  for (int K = 0; K < 4; ++K) {
    ck[K] = pcoef<T>(ch, 0, K) * rv[0] + pcoef<T>(ch, 1, K) * rv[1] + pcoef<T>(ch, 2, K) * rv[2] +
            pcoef<T>(ch, 3, K) * rv[3];
    ck[K] += __shfl_xor(ck[K], 16, 64);
    ck[K] += __shfl_xor(ck[K], 32, 64);
  }
  if (ch == 0) st4(a.rc + at(E, c), ck);
}

// Exact coarsest solve for kBatch requests, z = L_1^{-1} f in FP64: the
// 1024 x 1024 inverse times the 1024 x kBatch right-hand sides with FP64
// MFMA.  Workgroup R owns rows 16 R .. 16 R + 15; wavefront w the quarter
// 256 w .. 256 w + 255 of the contraction, summed in LDS in wavefront order.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_coarse_b(const double* __restrict__ inv,
                                                       const T* __restrict__ f, T* __restrict__ z) {
  using V = Mfma<double>::v4;
  __shared__ double red[4][4][64];
  const int R = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, k = lane >> 4;
  const double* ir = inv + (int64_t)(16 * R + r) * kCoarse + 4 * k;
  V acc = {0.0, 0.0, 0.0, 0.0};
  for (int g = 16 * wave; g < 16 * wave + 16; ++g) {   // contraction dofs 16 g .. 16 g + 15
    double av[4];
    ld4(ir + 16 * g, av);
    T bv[4];
    ld4(f + at(4 * g + k, r), bv);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) acc = Mfma<double>::mac(av[kk], static_cast<double>(bv[kk]), acc);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][v][lane] = acc[v];
  __syncthreads();
  if (wave == 0) {
    // rows 4 v + k of the block: square 4 R + v, corner k, request r
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double s = ((red[0][v][lane] + red[1][v][lane]) + red[2][v][lane]) + red[3][v][lane];
      z[at(4 * R + v, r) + k] = static_cast<T>(s);
    }
  }
}

// z = A f for kBatch columns, A dense FP64 m x m: workgroup R owns rows 16 R ..
// 16 R + 15, wavefront w of 8 an eighth of the contraction in FP64 MFMA steps,
// summed in LDS in wavefront order.  Bound by the matrix (134 MB at m = 4096) and
// the loads' latency, hence four groups of 16 columns' loads in flight.
constexpr int kFoldWaves = 8;
template <typename T>
__global__ __launch_bounds__(64 * kFoldWaves) void k_fold_b(int m, const double* __restrict__ A,
                                                            const T* __restrict__ f, T* __restrict__ z) {
  using V = Mfma<double>::v4;
  __shared__ double red[kFoldWaves][4][64];
  const int R = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, k = lane >> 4;
  const double* ir = A + (int64_t)(16 * R + r) * m + 4 * k;
  V acc = {0.0, 0.0, 0.0, 0.0}, acc1 = acc;
  const int per = m / 16 / kFoldWaves, g0 = per * wave;
  for (int g = g0; g < g0 + per; g += 4) {   // contraction dofs 16 g .. 16 g + 63
    double av[4][4];
    T bv[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ld4(ir + 16 * (g + u), av[u]);
      ld4(f + at(4 * (g + u) + k, r), bv[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc = Mfma<double>::mac(av[u][0], static_cast<double>(bv[u][0]), acc);
      acc1 = Mfma<double>::mac(av[u][1], static_cast<double>(bv[u][1]), acc1);
      acc = Mfma<double>::mac(av[u][2], static_cast<double>(bv[u][2]), acc);
      acc1 = Mfma<double>::mac(av[u][3], static_cast<double>(bv[u][3]), acc1);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][v][lane] = acc[v] + acc1[v];
  __syncthreads();
  if (wave < 4) {   // wavefront v: rows 4 v + k of the block: square 4 R + v, corner k
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kFoldWaves; ++w) s += red[w][wave][lane];
    z[at(4 * R + wave, r) + k] = static_cast<T>(s);
  }
}

__global__ __launch_bounds__(kThreads) void k_unit_columns(int ne, int j0, double* __restrict__ f) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= 4 * (int64_t)B * ne) return;
  const int64_t e = i / (4 * B);
  const int c = int((i >> 2) % B), j = int(i & 3);
  f[i] = 4 * e + j == j0 + c ? 1.0 : 0.0;
}

__global__ __launch_bounds__(kThreads) void k_store_columns(int ne, int j0, int has_z,
                                                            const double* __restrict__ z,
                                                            const double* __restrict__ Ye,
                                                            double* __restrict__ A) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= 4 * (int64_t)B * ne) return;
  const int64_t row = i / B, e = row >> 2;
  const int c = int(i % B), j = int(row & 3);
  double v = has_z ? z[at(e, c) + j] : 0.0;
  if (Ye) v = ((v + Ye[at(3 * e, c) + j]) + Ye[at(3 * e + 1, c) + j]) + Ye[at(3 * e + 2, c) + j];
  A[row * 4 * ne + j0 + c] = v;
}

// out = (has_z ? z : 0) + pending Ye for kBatch requests.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_resolve_b(int ne, int has_z, const T* __restrict__ z,
                                                        const T* __restrict__ Ye,
                                                        T* __restrict__ out) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= 4 * (int64_t)B * ne) return;
  const int64_t e = i / (4 * B);
  const int c = int((i >> 2) % B), j = int(i & 3);
  const T v = has_z ? z[i] : T(0);
  out[i] = ((v + Ye[at(3 * e, c) + j]) + Ye[at(3 * e + 1, c) + j]) + Ye[at(3 * e + 2, c) + j];
}

}  // namespace

template <typename T>
hipError_t launch_resolve_b(int ne, bool has_z, const T* z, const T* Ye, T* out, hipStream_t st) {
  const int64_t n = 4 * (int64_t)B * ne;
  k_resolve_b<T><<<int((n + kThreads - 1) / kThreads), kThreads, 0, st>>>(ne, has_z, z, Ye, out);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fold_b(int m, const double* A, const T* f, T* z, hipStream_t st) {
  if (m <= 0 || m % (64 * kFoldWaves)) return hipErrorInvalidValue;
  k_fold_b<T><<<m / 16, 64 * kFoldWaves, 0, st>>>(m, A, f, z);
  return hipGetLastError();
}

hipError_t launch_unit_columns(int ne, int j0, double* f, hipStream_t st) {
  const int64_t n = 4 * (int64_t)B * ne;
  k_unit_columns<<<int((n + kThreads - 1) / kThreads), kThreads, 0, st>>>(ne, j0, f);
  return hipGetLastError();
}

hipError_t launch_store_columns(int ne, int j0, bool has_z, const double* z, const double* Ye, double* A,
                                hipStream_t st) {
  const int64_t n = 4 * (int64_t)B * ne;
  k_store_columns<<<int((n + kThreads - 1) / kThreads), kThreads, 0, st>>>(ne, j0, has_z, z, Ye, A);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_sweep_b(const SweepArgs<T>& a, hipStream_t st) {
  const int tpr = a.n / 4;
  if (a.tiles <= 0 || a.n < 8 || (a.n & 3) || a.tiles != tpr * tpr) return hipErrorInvalidValue;
#define DCG_SWEEP_B(NW, NS)                                                    \
  if (a.prol)                                                                  \
    k_sweep_b<T, true, NW, NS><<<NS * a.tiles, 64 * NW, 0, st>>>(a);           \
  else                                                                         \
    k_sweep_b<T, false, NW, NS><<<NS * a.tiles, 64 * NW, 0, st>>>(a)
  // up to one workgroup per compute unit 8 wavefronts each, see the kernel
  if (4 * a.tiles <= 256) { DCG_SWEEP_B(8, 4); }
  else if (a.tiles <= 256) { DCG_SWEEP_B(8, 1); }
  else { DCG_SWEEP_B(4, 1); }
#undef DCG_SWEEP_B
  return hipGetLastError();
}

template <typename T>
hipError_t launch_restrict_res_b(const RestrictArgs<T>& a, hipStream_t st) {
  const int nc = a.n / 2;
  k_restrict_res_b<T><<<(nc * nc + 3) / 4, kThreads, 0, st>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_coarse_b(const double* inv, const T* f, T* z, hipStream_t st) {
  k_coarse_b<T><<<kCoarse / 16, kThreads, 0, st>>>(inv, f, z);
  return hipGetLastError();
}

#define DCG_MGB_INSTANTIATE(T)                                                              \
  template hipError_t launch_sweep_b<T>(const SweepArgs<T>&, hipStream_t);                  \
  template hipError_t launch_restrict_res_b<T>(const RestrictArgs<T>&, hipStream_t);        \
  template hipError_t launch_coarse_b<T>(const double*, const T*, T*, hipStream_t);       \
  template hipError_t launch_fold_b<T>(int, const double*, const T*, T*, hipStream_t);     \
  template hipError_t launch_resolve_b<T>(int, bool, const T*, const T*, T*, hipStream_t);

DCG_MGB_INSTANTIATE(float)
DCG_MGB_INSTANTIATE(double)

}  // namespace dcg

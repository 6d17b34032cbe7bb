// Device side of the exact inner solve by fast diagonalisation (2D path):
// z = L^{-1} s = V' diag(1 / (lam_y + lam_x)) V'^T s with V' = V (x) V on the
// tensor index (Iy, Ix), applied as four dense N x N products (N = 2 n):
//   T1 = S V,  T2 = (V^T T1) ./ (lam_i + lam_k),  T3 = V T2,  Z = T3 V^T,
// with S, Z the scalar vectors rearranged from the element-major layout
// 4 e + j (e = ey n + ex, j = ix + 2 iy) to the row-major tensor (Iy, Ix),
// Ix = 2 ex + ix.  The products are FP64 MFMA GEMMs staged through LDS.  The
// same solve serves as the exact coarsest-level solve of a shortened
// multigrid hierarchy, whose level vectors may be FP32.
#include <cstdint>

#include "kernels.hpp"
#include "mg_common.hpp"

namespace dcg {
namespace {

constexpr int kGThreads = 512;

// Position of tensor entry (Iy, Ix) in the element-major layout.
__device__ __forceinline__ int64_t tensor_to_elem(int n, int a, int c) {
  return 4 * ((int64_t)(a >> 1) * n + (c >> 1)) + (c & 1) + 2 * (a & 1);
}

// C = A B (+ D), N x N row-major FP64; with la: (A B)[i][k] is multiplied
// by 1 / (la[i] + lb[k]).
// AELEM: A is an element-major vector (of type TIN);
// CELEM: C is written element-major (as TOUT), so the layout changes need no
// launches of their own.  One TILE x TILE block of C per workgroup; two groups
// of 4 wavefronts take half of every K-slab each, a wavefront (TILE / 2)^2 outputs
// in 16 x 16 x 4 MFMA tiles, so that a SIMD has a second wavefront to issue from
// while one reads its operands.  K-slabs of KK are double-buffered in LDS with
// the next slab's loads in flight (registers) during the products.
// The LDS strides spread an operand's 64 values evenly over the banks.  N is a
// multiple of TILE and KK.
// Bound by the FP64 matrix rate: at N = 1024 a product takes 50 us, 43 TFLOP/s
// (126 us with vector FMAs, 2 x 2 outputs a thread).
template <int TILE, int KK, bool AELEM, bool CELEM, typename TIN, typename TOUT>
__global__ __launch_bounds__(kGThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm(int N, const TIN* __restrict__ A,
                                                    const double* __restrict__ B, TOUT* __restrict__ C,
                                                    const double* __restrict__ la,
                                                    const double* __restrict__ lb,
                                                    const double* D) {
  using V = mg::Mfma<double>::v4;
  constexpr int SA = KK + 2, SB = TILE + 16, R = TILE / 32, NL = TILE * KK / (2 * kGThreads);
  __shared__ __align__(16) double As[2][TILE * SA];   // As[row][k]
  __shared__ __align__(16) double Bs[2][KK * SB];     // Bs[k][col]
  const int tid = threadIdx.x, lane = tid & 63, w = (tid >> 6) & 3, half = tid >> 8;
  const int row0 = blockIdx.y * TILE, col0 = blockIdx.x * TILE;
  const int wr = (w >> 1) * 16 * R, wc = (w & 1) * 16 * R;
  const int n = N >> 1;
  // the slab in flight (vectors, which stay in registers where arrays written
  // under a condition went through LDS)
  typedef double slab_t __attribute__((ext_vector_type(4)));
  static_assert(NL == 2, "two 16-byte loads of A and of B per thread and slab");
  slab_t ra, rb;
  auto fetch = [&](int k0) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int t = tid + u * kGThreads;
      const int r = t / (KK / 2), kk = 2 * (t % (KK / 2));        // A: row r, columns kk, kk + 1
      const TIN* a = A + (AELEM ? tensor_to_elem(n, row0 + r, k0 + kk) : (int64_t)(row0 + r) * N + k0 + kk);
      ra[2 * u] = double(a[0]);
      ra[2 * u + 1] = double(a[1]);
      const int kb = t / (TILE / 2), c = 2 * (t % (TILE / 2));    // B: row kb, columns c, c + 1
      const double2 bv = *reinterpret_cast<const double2*>(B + (int64_t)(k0 + kb) * N + col0 + c);
      rb[2 * u] = bv.x;
      rb[2 * u + 1] = bv.y;
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int t = tid + u * kGThreads;
      const int r = t / (KK / 2), kk = 2 * (t % (KK / 2));
      *reinterpret_cast<double2*>(&As[buf][r * SA + kk]) = make_double2(ra[2 * u], ra[2 * u + 1]);
      const int kb = t / (TILE / 2), c = 2 * (t % (TILE / 2));
      *reinterpret_cast<double2*>(&Bs[buf][kb * SB + c]) = make_double2(rb[2 * u], rb[2 * u + 1]);
    }
  };
  V acc[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[i][j] = V{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  stage(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < N; k0 += KK, buf ^= 1) {
    const bool more = k0 + KK < N;
    if (more) fetch(k0 + KK);
    const double* ap = &As[buf][(wr + (lane & 15)) * SA + (lane >> 4) + half * (KK / 2)];
    const double* bp = &Bs[buf][((lane >> 4) + half * (KK / 2)) * SB + wc + (lane & 15)];
#pragma unroll
    for (int k = 0; k < KK / 2; k += 4) {
      double a[R], b[R];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        a[i] = ap[16 * i * SA + k];
        b[i] = bp[k * SB + 16 * i];
      }
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j) acc[i][j] = mg::Mfma<double>::mac(a[i], b[j], acc[i][j]);
    }
    if (more) stage(buf ^ 1);   // last read before the previous barrier
    __syncthreads();
  }
  // the other half of the contraction, through LDS
  double* red = &Bs[0][0];
  static_assert(2 * KK * SB >= TILE * TILE, "the partial tile fits the B slabs");
  if (half) {
#pragma unroll
    for (int i = 0; i < R * R; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[((i * 4 + v) * 4 + w) * 64 + lane] = acc[i / R][i % R][v];
  }
  __syncthreads();
  if (half) return;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int gr = row0 + wr + 16 * i + 4 * v + (lane >> 4), gc = col0 + wc + 16 * j + (lane & 15);
        double x = acc[i][j][v] + red[(((i * R + j) * 4 + v) * 4 + w) * 64 + lane];
        if (la) x *= 1.0 / (la[gr] + lb[gc]);
        if (D) x += D[(int64_t)gr * N + gc];
        C[CELEM ? tensor_to_elem(n, gr, gc) : (int64_t)gr * N + gc] = TOUT(x);
      }
}

template <bool AELEM, bool CELEM, typename TIN, typename TOUT>
hipError_t gemm(int N, const TIN* A, const double* B, TOUT* C, const double* la, const double* lb,
                hipStream_t st, const double* D = nullptr) {
  // 64 x 64 tiles fill the compute units from N = 1024 on (256 workgroups);
  // below, 32 x 32 tiles do
  if (N % 64) return hipErrorInvalidValue;
  if (N >= 1024)
    k_gemm<64, 32, AELEM, CELEM><<<dim3(N / 64, N / 64), kGThreads, 0, st>>>(N, A, B, C, la, lb, D);
  else
    k_gemm<32, 64, AELEM, CELEM><<<dim3(N / 32, N / 32), kGThreads, 0, st>>>(N, A, B, C, la, lb, D);
  return hipGetLastError();
}

// Small grids (N = 2 n in {32, 64, 128}: coarse levels) in two passes
// with the layout change folded into the loads and stores, one workgroup per
// row:
//   forward:  T2[i][k] = (sum_a sum_c V[a][i] S[a][c] V[c][k]) / (lam_i + lam_k),
//             row i of U = V^T S, then of U V;
//   backward: Z[a][c] = sum_i sum_k V[a][i] T2[i][k] V[c][k],
//             row a of W = V T2, then of W V^T.
// Thread t forms a partial sum for column t % N over the contraction range
// [p LEN, (p + 1) LEN), p = t / N; the P partials of a column are added in
// LDS in ascending p (fixed order).  A workgroup reads two N x N matrices for 4 N^2
// flop, so the passes are bound by one round of loads: both products' operands are
// requested at the start, N / 8 per thread and product.  At N = 128 / 64 / 32 a pass
// takes 6.7 / 3.5 / 2.7 us (7.7 / 4.2 / 4.3 with 256 threads that loaded one product's
// operands after the other).  At N = 256 the two matrices are 1 MB through one
// compute unit's cache: 19 us a pass, 38 for the solve, against 24 as four products below.
template <int N>
struct FdmRows {
  static constexpr int P = 8, LEN = N / P, threads = N * P;
};

// sum over p of part[p N + c] for the threads t < N (column c = t)
template <int N>
__device__ __forceinline__ double column_total(const double* part, int c) {
  double t = 0.0;
#pragma unroll
  for (int p = 0; p < FdmRows<N>::P; ++p) t += part[p * N + c];
  return t;
}

template <int N, bool FWD, typename TIN, typename TOUT>
__global__ __launch_bounds__(FdmRows<N>::threads) void k_fdm_row(const double* __restrict__ V,
                                                                 const double* __restrict__ VT,
                                                                 const double* __restrict__ lam,
                                                                 const TIN* __restrict__ in,
                                                                 TOUT* __restrict__ out) {
  using F = FdmRows<N>;
  constexpr int n = N / 2;
  __shared__ double lhs[N], mid[N], part[F::threads];
  const int tid = threadIdx.x, c = tid % N, q0 = (tid / N) * F::LEN, row = blockIdx.x;
  const double* M = (FWD ? V : VT) + (int64_t)q0 * N + c;   // the second product's matrix
  double b1[F::LEN], b2[F::LEN];
#pragma unroll
  for (int j = 0; j < F::LEN; ++j)
    b1[j] = FWD ? double(in[tensor_to_elem(n, q0 + j, c)]) : double(in[(int64_t)(q0 + j) * N + c]);
#pragma unroll
  for (int j = 0; j < F::LEN; ++j) b2[j] = M[(int64_t)j * N];
  if (tid < N) lhs[tid] = (FWD ? VT : V)[(int64_t)row * N + tid];
  __syncthreads();
  double u = 0.0;
#pragma unroll
  for (int j = 0; j < F::LEN; ++j) u += lhs[q0 + j] * b1[j];
  part[tid] = u;
  __syncthreads();
  if (tid < N) mid[tid] = column_total<N>(part, tid);
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int j = 0; j < F::LEN; ++j) t += mid[q0 + j] * b2[j];
  part[tid] = t;
  __syncthreads();
  if (tid >= N) return;
  const double x = column_total<N>(part, tid);
  if (FWD) out[(int64_t)row * N + tid] = TOUT(x * (1.0 / (lam[row] + lam[tid])));
  else out[tensor_to_elem(n, row, tid)] = TOUT(x);
}

template <int N, typename T>
hipError_t fdm_rows(const double* V, const double* VT, const double* lam, const T* s, T* z, double* t,
                    hipStream_t st) {
  k_fdm_row<N, true, T, double><<<N, FdmRows<N>::threads, 0, st>>>(V, VT, lam, s, t);
  k_fdm_row<N, false, double, T><<<N, FdmRows<N>::threads, 0, st>>>(V, VT, lam, t, z);
  return hipGetLastError();
}

template <typename T>
hipError_t fdm_solve(int n, const double* V, const double* VT, const double* lam, const T* s, T* z,
                     double* t0, double* t1, double* t2, hipStream_t st) {
  const int N = 2 * n;
  switch (N) {
    case 32: return fdm_rows<32, T>(V, VT, lam, s, z, t0, st);
    case 64: return fdm_rows<64, T>(V, VT, lam, s, z, t0, st);
    case 128: return fdm_rows<128, T>(V, VT, lam, s, z, t0, st);
    default: break;
  }
  hipError_t e = gemm<true, false>(N, s, V, t1, nullptr, nullptr, st);                      // x: S V
  if (e != hipSuccess) return e;
  if ((e = gemm<false, false>(N, VT, t1, t2, lam, lam, st)) != hipSuccess) return e;        // y: V^T T1, scaled
  if ((e = gemm<false, false>(N, V, t2, t0, nullptr, nullptr, st)) != hipSuccess) return e;  // y: V T2
  return gemm<false, true>(N, t0, VT, z, nullptr, nullptr, st);                             // x: T3 V^T
}

}  // namespace

hipError_t launch_gemm(int N, const double* A, const double* B, double* C, const double* D, hipStream_t st) {
  return gemm<false, false>(N, A, B, C, nullptr, nullptr, st, D);
}

hipError_t launch_fdm_solve2d(int n, const double* V, const double* VT, const double* lam,
                              const double* s, double* z, double* t0, double* t1, double* t2,
                              hipStream_t st) {
  return fdm_solve<double>(n, V, VT, lam, s, z, t0, t1, t2, st);
}

template <typename T>
hipError_t launch_fdm_coarse(int n, const double* V, const double* VT, const double* lam,
                             const T* f, T* z, double* t0, double* t1, double* t2, hipStream_t st) {
  return fdm_solve<T>(n, V, VT, lam, f, z, t0, t1, t2, st);
}

template hipError_t launch_fdm_coarse<float>(int, const double*, const double*, const double*,
                                             const float*, float*, double*, double*, double*,
                                             hipStream_t);
template hipError_t launch_fdm_coarse<double>(int, const double*, const double*, const double*,
                                              const double*, double*, double*, double*, double*,
                                              hipStream_t);

}  // namespace dcg

// Kernels of the three-dimensional deflated CG (the d = 3 block structure of
// Section 3.1; deflation as in Algorithm 2 with V of eq. (Vmatrix)).
//
// The A* product and the deflation correction run as FP64 MFMA products of the
// 24 x 24 blocks C_3, which are a table of the uniform grid, with the vectors
// of 16 elements a wavefront, and so does the exact inner solve by fast
// diagonalisation.  The iterative inner Laplace system (dt/3) L (Corollary 1, d = 3) is
// solved by block-Jacobi preconditioned CG whose scalars stay on the device;
// every reduction is a fixed-order two-stage sum, so results are
// reproducible bit for bit.
#include <cmath>

#include "dcg3d.hpp"
#include "mg_common.hpp"

namespace dcg3 {
namespace {

using dcg::mg::ld2_any;   // the caller's vectors
using dcg::mg::st2_any;

constexpr int kThreads = 256;
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kMaxPartials = 1024;

__device__ __forceinline__ int nbr3(int n, int e, int s) {
  const int ex = e % n, ey = (e / n) % n, ez = e / (n * n);
  switch (s) {
    case 0: return e;
    case 1: return ex > 0 ? e - 1 : -1;
    case 2: return ex + 1 < n ? e + 1 : -1;
    case 3: return ey > 0 ? e - n : -1;
    case 4: return ey + 1 < n ? e + n : -1;
    case 5: return ez > 0 ? e - n * n : -1;
    default: return ez + 1 < n ? e + n * n : -1;
  }
}

// Sum over the workgroup (kThreads threads, all participating); valid in
// thread 0.  Fixed order: butterfly within each wavefront, then the 4
// wavefront sums in order.
__device__ double block_sum(double v, double* lds) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[w] = v;
  __syncthreads();
  return ((lds[0] + lds[1]) + lds[2]) + lds[3];
}

// Sum of part[0 .. cnt) by one workgroup, fixed order.
__device__ double final_sum(const double* __restrict__ part, int cnt, double* lds) {
  double v = 0.0;
  for (int i = threadIdx.x; i < cnt; i += kThreads) v += part[i];
  return block_sum(v, lds);
}

// ---- A* and A_div Z as FP64 MFMA products.  On the uniform grid the block of
// a face neighbour does not depend on the element and the element's own block
// only on its class (which sides of the domain it touches, 27 classes), so
// C_3 is a table (build_astar_tiles) and not a stream: one wavefront takes 16
// consecutive elements as the columns and the tensor row k its B operand
// comes from, the 24 rows of C_3 are two 16-row tiles (a0: rows 0..15, a1:
// rows 16..23 and padding), and the blocks of a face normal to axis a that the
// form leaves zero (i != a and j != a, Section 3.3.2) are not multiplied.
// Column 8 t + 2 q + h of a 24-column block is step (t, h), lane group q, so
// that a lane's operands of one t are one 16-byte load; rows are permuted so
// that a lane's results are consecutive in memory.  Lanes outside the domain
// enter zeros; a wavefront whose elements are of several classes runs the 6
// steps of the own block once per class.
//
// With every block read from memory (1.07 GB a launch at n = 32, the HBM
// rate) the two products took 205 and 200 us; with the table 41 and 17 us,
// bound by the latency of the vector and table reads (12 us of matrix work).
__device__ __forceinline__ v4d mfma64(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int axis_class(int x, int n) { return x == 0 ? 0 : (x == n - 1 ? 2 : 1); }

// Class of element e; -1 outside the mesh.
__device__ __forceinline__ int elem_class(int n, int ne, int e) {
  if (e >= ne) return -1;
  return axis_class(e % n, n) + 3 * axis_class((e / n) % n, n) + 9 * axis_class(e / (n * n), n);
}

// Workgroup index with the 8 XCDs (dispatched round robin) on contiguous
// ranges of elements, so that the planes z +- 1 of a range stay in one L2.
__device__ __forceinline__ int band_index(int b, int G) {
  return (G & 7) ? b : (b & 7) * (G >> 3) + (b >> 3);
}

// G groups of 16 elements per workgroup, a wavefront per group and tensor row.
template <int G>
__global__ __launch_bounds__(G * 192) void k_astar3(int n, const double* __restrict__ At, double inv_nu,
                                                    double dt, const double* __restrict__ x,
                                                    double* __restrict__ y, double inv_sqrt3,
                                                    double* __restrict__ s) {
  __shared__ __align__(16) double tab[kFixedTiles * 64];
  __shared__ double zl[G * 16][3][kNb];
  const int ne = n * n * n;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = __builtin_amdgcn_readfirstlane(w % 3), grp = w / 3;
  const int col = lane & 15, q = lane >> 4;
  const int e = (band_index(blockIdx.x, gridDim.x) * G + grp) * 16 + col;
  const bool live = e < ne;
  double2 v[kSlots][3];
#pragma unroll
  for (int sl = 0; sl < kSlots; ++sl) {
    const int nb = live ? nbr3(n, e, sl) : -1;
    const double* p = x + (int64_t)(nb < 0 ? 0 : nb) * kDof + 24 * k + 2 * q;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      v[sl][t] = make_double2(0.0, 0.0);
      if (nb >= 0) v[sl][t] = ld2_any(p + 8 * t);
    }
  }
  // sigma_{k1 k1} + sigma_{k2 k2} of the other two rows, for the mass term
  const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
  const double* xe = x + (int64_t)(live ? e : 0) * kDof + 2 * q;
  const double2 o1 = ld2_any(xe + 32 * k1);
  const double2 o2 = ld2_any(xe + 32 * k2);
  constexpr int TT = G * 192, NS = (kFixedTiles * 32 + TT - 1) / TT;
  double2 tv[NS];
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int i = threadIdx.x + u * TT;
    tv[u] = reinterpret_cast<const double2*>(At)[i < kFixedTiles * 32 ? i : 0];
  }
  __builtin_amdgcn_sched_barrier(0);   // every load of the element is in flight
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int i = threadIdx.x + u * TT;
    if (i < kFixedTiles * 32) reinterpret_cast<double2*>(tab)[i] = tv[u];
  }
  __syncthreads();
  v4d a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0, m0 = a0, m1 = a0;
  int tile = 0;
#pragma unroll
  for (int sl = 1; sl < kSlots; ++sl) {
    const int ax = (sl - 1) >> 1;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double b = h ? v[sl][t].y : v[sl][t].x;
        if (t == ax || ax < 2) a0 = mfma64(tab[(tile++) * 64 + lane], b, a0);
        if (t == ax || ax == 2) a1 = mfma64(tab[(tile++) * 64 + lane], b, a1);
      }
  }
  // (C_9 (x) M_1) x on the element: off-diagonal components carry weight 1,
  // the diagonal ones 2/3 on themselves and -1/3 on the other two.
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      double b = h ? v[0][t].y : v[0][t].x;
      if (t == k) b = (2.0 / 3.0) * b - (1.0 / 3.0) * (h ? o1.y + o2.y : o1.x + o2.x);
      const double m = tab[(tile++) * 64 + lane];
      if (t < 2) m0 = mfma64(m, b, m0);
      else m1 = mfma64(m, b, m1);
    }
  // the element's own block, once per class in the wavefront
  const int cls = elem_class(n, ne, e);
  uint64_t pending = __ballot(live);
  while (pending) {
    const int c = __builtin_amdgcn_readfirstlane(__shfl(cls, __builtin_ctzll(pending), 64));
    const bool mine = cls == c;
    const double* S = At + ((int64_t)kFixedTiles + c * kSelfTiles) * 64 + lane;
    double a[kSelfTiles];
#pragma unroll
    for (int i = 0; i < kSelfTiles; ++i) a[i] = S[64 * i];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double b = mine ? (h ? v[0][t].y : v[0][t].x) : 0.0;
        a0 = mfma64(a[4 * t + 2 * h], b, a0);
        a1 = mfma64(a[4 * t + 2 * h + 1], b, a1);
      }
    pending &= ~__ballot(mine);
  }
  double r0[4], r1[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) r0[i] = inv_nu * m0[i] + dt * a0[i];
#pragma unroll
  for (int i = 0; i < 2; ++i) r1[i] = inv_nu * m1[i] + dt * a1[i];
  if (live) {   // rows 4 q .. 4 q + 3 and 16 + 2 q, 16 + 2 q + 1
    double* yp = y + (int64_t)e * kDof + 24 * k;
    st2_any(yp + 4 * q, r0[0], r0[1]);
    st2_any(yp + 4 * q + 2, r0[2], r0[3]);
    st2_any(yp + 16 + 2 * q, r1[0], r1[1]);
  }
  if (!s) return;
  // s = Z^T y: rows 8 k .. 8 k + 7 of the three tensor rows
  if (k < 2) {
    if ((q >> 1) == k)
#pragma unroll
      for (int i = 0; i < 4; ++i) zl[16 * grp + col][k][4 * (q & 1) + i] = r0[i];
  } else {
    zl[16 * grp + col][2][2 * q] = r1[0];
    zl[16 * grp + col][2][2 * q + 1] = r1[1];
  }
  __syncthreads();
  if (k == 0 && live) {
    const double(*z)[kNb] = zl[16 * grp + col];
    double2 sv;
    sv.x = ((z[0][2 * q] + z[1][2 * q]) + z[2][2 * q]) * inv_sqrt3;
    sv.y = ((z[0][2 * q + 1] + z[1][2 * q + 1]) + z[2][2 * q + 1]) * inv_sqrt3;
    *reinterpret_cast<double2*>(s + (int64_t)e * kNb + 2 * q) = sv;
  }
}

// q = w - dt A_div Z yh: the products of k_astar3 with the one column block
// t = k of C_3 that a multiple of the identity meets.
__global__ __launch_bounds__(192) void k_adivz3(int n, const double* __restrict__ At, double dt,
                                                double inv_sqrt3, const double* __restrict__ w,
                                                const double* __restrict__ yh, double* __restrict__ qv) {
  const int ne = n * n * n;
  const int lane = threadIdx.x & 63;
  const int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, q = lane >> 4;
  const int e = band_index(blockIdx.x, gridDim.x) * 16 + col;
  const bool live = e < ne;
  double2 v[kSlots];
#pragma unroll
  for (int sl = 0; sl < kSlots; ++sl) {
    const int nb = live ? nbr3(n, e, sl) : -1;
    const double2 yv = ld2_any(yh + (int64_t)(nb >= 0 ? nb : 0) * kNb + 2 * q);
    v[sl].x = nb >= 0 ? yv.x * inv_sqrt3 : 0.0;
    v[sl].y = nb >= 0 ? yv.y * inv_sqrt3 : 0.0;
  }
  double2 wv[3];
  const double* wp = w + (int64_t)(live ? e : 0) * kDof + 24 * k;
  wv[0] = ld2_any(wp + 4 * q);
  wv[1] = ld2_any(wp + 4 * q + 2);
  wv[2] = ld2_any(wp + 16 + 2 * q);
  v4d a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0;
#pragma unroll
  for (int sl = 1; sl < kSlots; ++sl) {
    const int ax = (sl - 1) >> 1;
    // first tile of (slot, t = k): two per step where t = axis, else one
    const double* T = At + ((sl - 1) * kSlotTiles + 2 * k + (k > ax ? 2 : 0)) * 64 + lane;
    if (k == ax) {
      a0 = mfma64(T[0], v[sl].x, a0);
      a1 = mfma64(T[64], v[sl].x, a1);
      a0 = mfma64(T[128], v[sl].y, a0);
      a1 = mfma64(T[192], v[sl].y, a1);
    } else if (ax < 2) {
      a0 = mfma64(T[0], v[sl].x, a0);
      a0 = mfma64(T[64], v[sl].y, a0);
    } else {
      a1 = mfma64(T[0], v[sl].x, a1);
      a1 = mfma64(T[64], v[sl].y, a1);
    }
  }
  const int cls = elem_class(n, ne, e);
  uint64_t pending = __ballot(live);
  while (pending) {
    const int c = __builtin_amdgcn_readfirstlane(__shfl(cls, __builtin_ctzll(pending), 64));
    const bool mine = cls == c;
    const double* S = At + ((int64_t)kFixedTiles + c * kSelfTiles + 4 * k) * 64 + lane;
    const double bx = mine ? v[0].x : 0.0, by = mine ? v[0].y : 0.0;
    a0 = mfma64(S[0], bx, a0);
    a1 = mfma64(S[64], bx, a1);
    a0 = mfma64(S[128], by, a0);
    a1 = mfma64(S[192], by, a1);
    pending &= ~__ballot(mine);
  }
  if (!live) return;
  double* op = qv + (int64_t)e * kDof + 24 * k;
  st2_any(op + 4 * q, wv[0].x - dt * a0[0], wv[0].y - dt * a0[1]);
  st2_any(op + 4 * q + 2, wv[1].x - dt * a0[2], wv[1].y - dt * a0[3]);
  st2_any(op + 16 + 2 * q, wv[2].x - dt * a1[0], wv[2].y - dt * a1[1]);
}

__global__ __launch_bounds__(kThreads) void k_zt3(int64_t ne, double inv_sqrt3,
                                                  const double* __restrict__ w, double* __restrict__ s) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= ne * kNb) return;
  const int64_t e = i >> 3;
  const int a = int(i & 7);
  const double* we = w + e * kDof + a;
  s[i] = ((we[0] + we[32]) + we[64]) * inv_sqrt3;
}

__global__ __launch_bounds__(kThreads) void k_zaxpy3(int64_t ne, double c, const double* __restrict__ y,
                                                     double* __restrict__ x) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= ne * kNb) return;
  const int64_t e = i >> 3;
  const int a = int(i & 7);
  const double v = c * y[i];
  double* xe = x + e * kDof + a;
  xe[0] += v;
  xe[32] += v;
  xe[64] += v;
}

__global__ __launch_bounds__(kThreads) void k_lap3(int n, const double* __restrict__ Ld, double scale,
                                                   const double* __restrict__ p, double* __restrict__ q,
                                                   double* __restrict__ part) {
  __shared__ double lds[4];
  const int ne = n * n * n;
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  double pq = 0.0;
  if (i < (int64_t)ne * kNb) {
    const int e = int(i >> 3), a = int(i & 7);
    double acc = 0.0;
    for (int s = 0; s < kSlots; ++s) {
      const int nb = nbr3(n, e, s);
      if (nb < 0) continue;
      const double* l = Ld + ((int64_t)s * ne + e) * 64 + a;
      const double* pn = p + (int64_t)nb * kNb;
#pragma unroll
      for (int b = 0; b < kNb; ++b) acc += l[8 * b] * pn[b];
    }
    const double v = scale * acc;
    q[i] = v;
    pq = p[i] * v;
  }
  pq = block_sum(pq, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = pq;
}

// z = Dinv r on the element of thread i (r of the element in LDS rl).
__device__ __forceinline__ double bj_apply(const double* __restrict__ Dinv, int64_t e, int a,
                                           const double* rl) {
  const double* d = Dinv + e * 64 + a;
  double z = 0.0;
#pragma unroll
  for (int b = 0; b < kNb; ++b) z += d[8 * b] * rl[b];
  return z;
}

__global__ __launch_bounds__(kThreads) void k_pcg_init(int64_t ne, const double* __restrict__ Dinv,
                                                       const double* __restrict__ s, double* __restrict__ x,
                                                       double* __restrict__ r, double* __restrict__ z,
                                                       double* __restrict__ p, double* __restrict__ part) {
  __shared__ double rl[kThreads];
  __shared__ double lds[4];
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  const bool live = i < ne * kNb;
  const double rv = live ? s[i] : 0.0;
  rl[threadIdx.x] = rv;
  __syncthreads();
  double rz = 0.0, rr = 0.0;
  if (live) {
    const double zv = bj_apply(Dinv, i >> 3, int(i & 7), rl + (threadIdx.x & ~7));
    x[i] = 0.0;
    r[i] = rv;
    z[i] = zv;
    p[i] = zv;
    rz = rv * zv;
    rr = rv * rv;
  }
  rz = block_sum(rz, lds);
  rr = block_sum(rr, lds);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = rz;
    part[gridDim.x + blockIdx.x] = rr;
  }
}

__global__ __launch_bounds__(kThreads) void k_pcg_init_final(const double* __restrict__ part, int cnt,
                                                             double rel2, PcgScalars* sc) {
  __shared__ double lds[4];
  const double rz = final_sum(part, cnt, lds);
  const double rr = final_sum(part + cnt, cnt, lds);
  if (threadIdx.x == 0) {
    sc->rho = rz;
    sc->rr = rr;
    sc->pq = 0.0;
    sc->alpha = sc->beta = 0.0;
    sc->thresh2 = rel2 * rr;
    sc->active = (rr > sc->thresh2 && rr > 0.0) ? 1 : 0;
    sc->iters = 0;
  }
}

__global__ __launch_bounds__(kThreads) void k_pcg_alpha(const double* __restrict__ part, int cnt,
                                                        PcgScalars* sc) {
  __shared__ double lds[4];
  const double pq = final_sum(part, cnt, lds);
  if (threadIdx.x == 0) {
    sc->pq = pq;
    if (sc->active && pq > 0.0 && std::isfinite(pq)) {
      sc->alpha = sc->rho / pq;
    } else {
      sc->alpha = 0.0;
      sc->active = 0;
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_pcg_update(int64_t ne, const double* __restrict__ Dinv,
                                                         double* __restrict__ x, double* __restrict__ r,
                                                         double* __restrict__ z, const double* __restrict__ p,
                                                         const double* __restrict__ q,
                                                         double* __restrict__ part,
                                                         const PcgScalars* sc) {
  __shared__ double rl[kThreads];
  __shared__ double lds[4];
  const double alpha = sc->alpha;
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  const bool live = i < ne * kNb;
  double rv = 0.0;
  if (live) {
    x[i] += alpha * p[i];
    rv = r[i] - alpha * q[i];
    r[i] = rv;
  }
  rl[threadIdx.x] = rv;
  __syncthreads();
  double rz = 0.0, rr = 0.0;
  if (live) {
    const double zv = bj_apply(Dinv, i >> 3, int(i & 7), rl + (threadIdx.x & ~7));
    z[i] = zv;
    rz = rv * zv;
    rr = rv * rv;
  }
  rz = block_sum(rz, lds);
  rr = block_sum(rr, lds);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = rz;
    part[gridDim.x + blockIdx.x] = rr;
  }
}

__global__ __launch_bounds__(kThreads) void k_pcg_beta(const double* __restrict__ part, int cnt,
                                                       PcgScalars* sc) {
  __shared__ double lds[4];
  const double rz = final_sum(part, cnt, lds);
  const double rr = final_sum(part + cnt, cnt, lds);
  if (threadIdx.x == 0) {
    if (sc->active) {
      sc->beta = rz / sc->rho;
      sc->rho = rz;
      sc->rr = rr;
      sc->iters += 1;
      if (!(rr > sc->thresh2)) sc->active = 0;
    } else {
      sc->beta = 0.0;
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_pcg_dir(int64_t len, const double* __restrict__ z,
                                                      double* __restrict__ p, const PcgScalars* sc) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i < len) p[i] = z[i] + sc->beta * p[i];
}

__global__ __launch_bounds__(kThreads) void k_dot_partial(int64_t len, const double* __restrict__ x,
                                                          const double* __restrict__ y,
                                                          double* __restrict__ part) {
  __shared__ double lds[4];
  double v = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < len;
       i += (int64_t)gridDim.x * kThreads)
    v += x[i] * y[i];
  v = block_sum(v, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = v;
}

__global__ __launch_bounds__(kThreads) void k_dot_final(const double* __restrict__ part, int cnt,
                                                        double* __restrict__ out) {
  __shared__ double lds[4];
  const double v = final_sum(part, cnt, lds);
  if (threadIdx.x == 0) out[0] = v;
}

__global__ __launch_bounds__(kThreads) void k_axpy(int64_t len, double a, const double* __restrict__ x,
                                                   double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i < len) y[i] += a * x[i];
}

__global__ __launch_bounds__(kThreads) void k_xpby(int64_t len, const double* __restrict__ x, double b,
                                                   double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i < len) y[i] = x[i] + b * y[i];
}

__global__ __launch_bounds__(kThreads) void k_fill(int64_t len, double v, double* __restrict__ x) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i < len) x[i] = v;
}

// ---- exact inner solve by fast diagonalisation: three launches of FP64 MFMA
// products on the N^3 tensor (N = 2 n), layout (Iz N + Iy) N + Ix, element-
// major 8 e + a at the ends:
//   k_fdm_plane  per plane Iz and chunk of 16 columns: U = S Bx, then Ay U
//   k_fdm_z      per 16 lines along z: U = Vz^T S scaled, then Vz U
// so each launch holds its intermediate in LDS and a workgroup's two products
// share one 16-column chunk.  A workgroup of 4 wavefronts gives each the row
// tiles w, w + 4, ..; column 8 t + 2 q + h of a contraction is step (t, h),
// lane group q.  (Six passes of one thread per output took 10-13 us each at
// n = 32, bound by their 64-step chain of table loads; the three launches
// take 8.0-8.7 us each.)
constexpr int kFdmThreads = 256;
constexpr int kFdmMaxN = 128;
constexpr int kFdmPad = 17;                // LDS row of 16 columns

constexpr int kFdmTrip = 4;                // steps of 8 whose loads are issued together

// out[m][c] = sum_k A(m, k) U[k][c] for the wavefront's row tiles; A is N x N
// row-major, U in LDS (rows up to the next multiple of 32 are zero-filled).
template <typename Store>
__device__ __forceinline__ void fdm_rows(int N, const double* __restrict__ A, const double* U, Store store) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = lane & 15, q = lane >> 4;
  for (int m0 = 16 * w; m0 < N; m0 += 64) {
    const int row = m0 + col;
    const double* Ar = A + (int64_t)(row < N ? row : 0) * N + 2 * q;
    v4d acc = {0.0, 0.0, 0.0, 0.0}, acc1 = acc;
    for (int k0 = 0; k0 < N; k0 += 8 * kFdmTrip) {
      double2 a[kFdmTrip];
#pragma unroll
      for (int u = 0; u < kFdmTrip; ++u) {
        a[u] = make_double2(0.0, 0.0);
        if (row < N && k0 + 8 * u + 2 * q < N) a[u] = *reinterpret_cast<const double2*>(Ar + k0 + 8 * u);
      }
#pragma unroll
      for (int u = 0; u < kFdmTrip; ++u) {
        acc = mfma64(a[u].x, U[(k0 + 8 * u + 2 * q) * kFdmPad + col], acc);
        acc1 = mfma64(a[u].y, U[(k0 + 8 * u + 2 * q + 1) * kFdmPad + col], acc1);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) store(m0 + 4 * v + q, acc[v] + acc1[v]);
  }
}

// Rows [N, next multiple of 32) of U: the padding of a contraction over N rows.
__device__ __forceinline__ void fdm_pad_rows(int N, double* U) {
  for (int i = threadIdx.x; i < (((N + 31) & ~31) - N) * 16; i += kFdmThreads)
    U[(N + i / 16) * kFdmPad + i % 16] = 0.0;
}

template <bool IN_ELEM, bool OUT_ELEM>
__global__ __launch_bounds__(kFdmThreads) void k_fdm_plane(int n, const double* __restrict__ Bx,
                                                           const double* __restrict__ Ay,
                                                           const double* __restrict__ in,
                                                           double* __restrict__ out) {
  __shared__ double U[kFdmMaxN * kFdmPad];
  const int N = 2 * n;
  const int Iz = blockIdx.y, c0 = 16 * blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = lane & 15, q = lane >> 4;
  const int c = c0 + col;
  // element-major position of (Ix, Iy) in this plane
  const int64_t ez = (int64_t)(Iz >> 1) * n * n;
  auto elem = [&](int Ix, int Iy) {
    return 8 * (ez + (int64_t)(Iy >> 1) * n + (Ix >> 1)) + (Ix & 1) + 2 * (Iy & 1) + 4 * (Iz & 1);
  };
  for (int m0 = 16 * w; m0 < N; m0 += 64) {
    const int row = m0 + col;              // Iy of the A operand
    v4d acc = {0.0, 0.0, 0.0, 0.0}, acc1 = acc;
    for (int k0 = 0; k0 < N; k0 += 8 * kFdmTrip) {
      double2 a[kFdmTrip];
      double b0[kFdmTrip], b1[kFdmTrip];
#pragma unroll
      for (int u = 0; u < kFdmTrip; ++u) {
        const int kk = k0 + 8 * u + 2 * q;
        a[u] = make_double2(0.0, 0.0);
        b0[u] = b1[u] = 0.0;
        if (kk < N) {
          if (row < N)
            a[u] = ld2_any(in + (IN_ELEM ? elem(kk, row) : ((int64_t)Iz * N + row) * N + kk));
          if (c < N) {
            b0[u] = Bx[(int64_t)kk * N + c];
            b1[u] = Bx[(int64_t)(kk + 1) * N + c];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kFdmTrip; ++u) {
        acc = mfma64(a[u].x, b0[u], acc);
        acc1 = mfma64(a[u].y, b1[u], acc1);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int Iy = m0 + 4 * v + q;
      if (Iy < N) U[Iy * kFdmPad + col] = acc[v] + acc1[v];
    }
  }
  fdm_pad_rows(N, U);
  __syncthreads();
  fdm_rows(N, Ay, U, [&](int Iy, double v) {
    if (Iy < N && c < N) out[OUT_ELEM ? elem(c, Iy) : ((int64_t)Iz * N + Iy) * N + c] = v;
  });
}

// t[.][j] <- Vz (scale / (lx + ly + lz)) Vz^T t[.][j] for the 16 lines j = Iy N + Ix
// of the workgroup (in place: a workgroup reads and writes its own lines only).
__global__ __launch_bounds__(kFdmThreads) void k_fdm_z(int n, const double* __restrict__ V,
                                                       const double* __restrict__ VT,
                                                       const double* __restrict__ lx,
                                                       const double* __restrict__ ly, double scale,
                                                       double* __restrict__ t) {
  __shared__ double S[kFdmMaxN * kFdmPad];
  __shared__ double U[kFdmMaxN * kFdmPad];
  const int N = 2 * n;
  const int64_t NN = (int64_t)N * N;
  const int64_t j0 = 16 * (int64_t)blockIdx.x;
  const int col = threadIdx.x & 15;
  const int64_t j = j0 + col;
  const bool live = j < NN;
  for (int k = threadIdx.x >> 4; k < N; k += kFdmThreads / 16)
    S[k * kFdmPad + col] = live ? t[k * NN + j] : 0.0;
  fdm_pad_rows(N, S);
  const double lxy = live ? lx[j % N] + ly[j / N] : 0.0;
  __syncthreads();
  fdm_rows(N, VT, S, [&](int Iz, double v) {
    if (Iz < N) U[Iz * kFdmPad + col] = live ? v * (scale / (lxy + ly[Iz])) : 0.0;
  });
  fdm_pad_rows(N, U);
  __syncthreads();
  fdm_rows(N, V, U, [&](int Iz, double v) {
    if (Iz < N && live) t[Iz * NN + j] = v;
  });
}

int blocks_for(int64_t len) { return int((len + kThreads - 1) / kThreads); }

const double kInvSqrt3 = 1.0 / std::sqrt(3.0);

}  // namespace

int partial_blocks(int64_t len) {
  const int64_t b = (len + kThreads - 1) / kThreads;
  return int(b < kMaxPartials ? (b > 0 ? b : 1) : kMaxPartials);
}

hipError_t launch_astar3(int n, const double* At, double inv_nu, double dt, const double* x, double* y,
                         double* s, hipStream_t st) {
  const int64_t groups = ((int64_t)n * n * n + 15) / 16;
  // two groups per workgroup share the 27 KB table; on small meshes one, to
  // put a workgroup on more compute units
  if (groups >= 512) {
    const unsigned grid = unsigned(((groups + 1) / 2 + 7) & ~int64_t(7));
    k_astar3<2><<<grid, 384, 0, st>>>(n, At, inv_nu, dt, x, y, kInvSqrt3, s);
  } else {
    k_astar3<1><<<unsigned(groups), 192, 0, st>>>(n, At, inv_nu, dt, x, y, kInvSqrt3, s);
  }
  return hipGetLastError();
}

hipError_t launch_adivz3(int n, const double* At, double dt, const double* w, const double* yh,
                         double* q, hipStream_t st) {
  const int64_t groups = ((int64_t)n * n * n + 15) / 16;
  k_adivz3<<<unsigned((groups + 7) & ~int64_t(7)), 192, 0, st>>>(n, At, dt, kInvSqrt3, w, yh, q);
  return hipGetLastError();
}

hipError_t launch_zt3(int64_t ne, const double* w, double* s, hipStream_t st) {
  k_zt3<<<blocks_for(ne * kNb), kThreads, 0, st>>>(ne, kInvSqrt3, w, s);
  return hipGetLastError();
}

hipError_t launch_zaxpy3(int64_t ne, double a, const double* y, double* x, hipStream_t st) {
  k_zaxpy3<<<blocks_for(ne * kNb), kThreads, 0, st>>>(ne, a * kInvSqrt3, y, x);
  return hipGetLastError();
}

hipError_t launch_lap3(int n, const double* Ld, double scale, const double* p, double* q,
                       double* part, hipStream_t st) {
  const int64_t ne = (int64_t)n * n * n;
  k_lap3<<<blocks_for(ne * kNb), kThreads, 0, st>>>(n, Ld, scale, p, q, part);
  return hipGetLastError();
}

hipError_t launch_pcg_start(int64_t ne, const double* Dinv, const double* s, double* x, double* r,
                            double* z, double* p, double* part, PcgScalars* sc, double rel2,
                            hipStream_t st) {
  const int g = blocks_for(ne * kNb);
  k_pcg_init<<<g, kThreads, 0, st>>>(ne, Dinv, s, x, r, z, p, part);
  k_pcg_init_final<<<1, kThreads, 0, st>>>(part, g, rel2, sc);
  return hipGetLastError();
}

hipError_t launch_pcg_step(int64_t ne, const double* Dinv, double* x, double* r, double* z,
                           double* p, const double* q, double* part, double* part2, int nblk_q,
                           PcgScalars* sc, hipStream_t st) {
  const int g = blocks_for(ne * kNb);
  k_pcg_alpha<<<1, kThreads, 0, st>>>(part, nblk_q, sc);
  k_pcg_update<<<g, kThreads, 0, st>>>(ne, Dinv, x, r, z, p, q, part2, sc);
  k_pcg_beta<<<1, kThreads, 0, st>>>(part2, g, sc);
  k_pcg_dir<<<g, kThreads, 0, st>>>(ne * kNb, z, p, sc);
  return hipGetLastError();
}

hipError_t launch_fdm_solve(int n, const double* Vx, const double* VxT, const double* Vy,
                            const double* VyT, const double* lx, const double* ly, double scale,
                            const double* in, double* out, double* t, hipStream_t st) {
  const int N = 2 * n;
  if (N > kFdmMaxN) return hipErrorInvalidValue;
  const dim3 planes((N + 15) / 16, N);
  k_fdm_plane<true, false><<<planes, kFdmThreads, 0, st>>>(n, Vx, VyT, in, t);
  k_fdm_z<<<unsigned(((int64_t)N * N + 15) / 16), kFdmThreads, 0, st>>>(n, Vy, VyT, lx, ly, scale, t);
  k_fdm_plane<false, true><<<planes, kFdmThreads, 0, st>>>(n, VxT, Vy, t, out);
  return hipGetLastError();
}

hipError_t launch_dot(int64_t len, const double* x, const double* y, double* part, double* out,
                      hipStream_t st) {
  const int g = partial_blocks(len);
  k_dot_partial<<<g, kThreads, 0, st>>>(len, x, y, part);
  k_dot_final<<<1, kThreads, 0, st>>>(part, g, out);
  return hipGetLastError();
}

hipError_t launch_axpy(int64_t len, double a, const double* x, double* y, hipStream_t st) {
  k_axpy<<<blocks_for(len), kThreads, 0, st>>>(len, a, x, y);
  return hipGetLastError();
}

hipError_t launch_xpby(int64_t len, const double* x, double b, double* y, hipStream_t st) {
  k_xpby<<<blocks_for(len), kThreads, 0, st>>>(len, x, b, y);
  return hipGetLastError();
}

hipError_t launch_fill(int64_t len, double v, double* x, hipStream_t st) {
  k_fill<<<blocks_for(len), kThreads, 0, st>>>(len, v, x);
  return hipGetLastError();
}

}  // namespace dcg3

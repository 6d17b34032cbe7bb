// gfx950 kernels of the deflated-CG hot path (paper Section 4, Algorithms 2-4).
//
// The operators of the uniform grid are tables (kernels.hpp), so the kernels stream
// vectors only.  Dot products are two-stage and deterministic: a fixed-order wave64
// shuffle tree and an LDS tree per workgroup, per-workgroup partials, and one
// fixed-order final pass (no floating-point atomics anywhere).
#include <hip/hip_ext.h>

#include "kernels.hpp"
#include "mg_common.hpp"

#include <cmath>

namespace dcg {
namespace {

constexpr int kThreads = 256;
constexpr double kInvSqrt2 = 0.70710678118654752440;

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Workgroup sum of v (all 256 threads participate); result valid in thread 0.
__device__ inline double block_sum(double v, double* lds) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) s = (lds[0] + lds[1]) + (lds[2] + lds[3]);
  return s;
}

using mg::ld4_any;   // 4-vector loads and stores: most vectors here can be a caller's
using mg::st4_any;

inline int grid_for(int64_t items, int per_block, int cap) {
  int64_t g = (items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  return int(g < cap ? g : cap);
}

// ============================================================ outer kernels
__device__ inline int slot_id(const Slots& sl) { return sl.list ? sl.list[blockIdx.y] : 0; }

// The value of the other lane of a pair (lanes 2 i, 2 i + 1).
__device__ __forceinline__ double pair_swap(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_update_dpp(0, int(uint32_t(b)), 0xB1, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, int(uint32_t(b >> 32)), 0xB1, 0xF, 0xF, true);
  return __builtin_bit_cast(double, uint64_t(uint32_t(lo)) | (uint64_t(uint32_t(hi)) << 32));
}

// acc += B u for a table block B (8 x 8, column-major, wave-uniform address):
// two columns of coefficients (32 scalar registers) at a time.
__device__ __forceinline__ void block_product(const double* __restrict__ B, const double (&u)[8],
                                              double (&acc)[8]) {
#pragma unroll
  for (int m = 0; m < 8; ++m) {
#pragma unroll
    for (int r = 0; r < 8; ++r) acc[r] += B[8 * m + r] * u[m];
    // keeps the next columns' scalar loads from being hoisted past the
    // scalar register file; vector memory may pass
    if (m & 1) __builtin_amdgcn_sched_barrier(0x30);
  }
}

// w = (1/nu) M u + dt A_div u, s = Z^T w.  Thread (square e, stress row k),
// lane pairs sharing a square: the 8 values of stress row k of a square are
// 64 contiguous bytes and meet the same 8 x 8 block C for both k (A_div =
// diag(C, C)).  On the uniform grid the block of a neighbour does not depend
// on the square and the own block only on its class, so the coefficients are
// the same for all lanes and come through the scalar cache, one of them feeding
// 64 products; a wavefront with squares of several classes runs the own block
// once per class.  M = C_dev (x) M_1 with C_dev the dev-dev coefficient matrix
// (Section 3.1): rows 11/22 see (u11 - u22)/2, rows 12/21 see u.
// At n = 1024 the plain product moves 268 MB in 76 us, 3.5 TB/s or 0.7 of a copy's
// rate, with the direction update at n = 512 143 MB in 48 us: a lane reads 64
// contiguous bytes of five squares at a 64-byte stride, so a wavefront's load touches
// four times the lines of a contiguous one.  With the blocks of every square read from
// memory the plain product took 159 us at n = 512 and 650 us at n = 1024 (HBM bound,
// 0.85 and 3.4 GB); now 29 and 76 us.
template <int MODE>
__global__ __launch_bounds__(kThreads) void k_astar(
    const double* __restrict__ Ct, int n, const double* __restrict__ x,
    const double* __restrict__ p_old, const double* __restrict__ b, const Scalars* __restrict__ sc,
    double* __restrict__ p_new, double* __restrict__ w, double* __restrict__ s,
    double* __restrict__ part, Slots sl) {
  __shared__ double lds[4];
  const int slot = slot_id(sl);
  x += slot * sl.tstride;
  if (p_old) p_old += slot * sl.tstride;
  if (b) b += slot * sl.tstride;
  if (p_new) p_new += slot * sl.tstride;
  if (w) w += slot * sl.tstride;
  if (s) s += slot * sl.sstride;
  sc += slot;
  if (part) part += slot * kSlotPart;
  const double dt = sc->dt, inv_nu = sc->inv_nu;
  const double beta = MODE == kAstarDir ? sc->beta : 0.0;
  const int ne = n * n;
  const int id = mg::xcd_band(blockIdx.x, gridDim.x) * kThreads + threadIdx.x;
  const int e = id >> 1, k = id & 1;
  const bool valid = e < ne;
  const int ex = e & (n - 1), ey = e / n;
  auto load = [&](int64_t i, bool ok, double (&u)[8]) {   // u of stress row i = 2 e + k
    if (ok) {
      ld4_any(x + 8 * i, u);
      ld4_any(x + 8 * i + 4, u + 4);
      if (MODE == kAstarDir) {
        double p[8];
        ld4_any(p_old + 8 * i, p);
        ld4_any(p_old + 8 * i + 4, p + 4);
#pragma unroll
        for (int m = 0; m < 8; ++m) u[m] += beta * p[m];
      }
    } else {
#pragma unroll
      for (int m = 0; m < 8; ++m) u[m] = 0.0;
    }
  };
  double u0[8], acc[8];
  load(id, valid, u0);
#pragma unroll
  for (int r = 0; r < 8; ++r) acc[r] = 0.0;
  {
    const int cls = square_class(ex, ey, n);
    uint64_t pending = __ballot(valid);
    while (pending) {
      const int c = __builtin_amdgcn_readlane(cls, __builtin_ctzll(pending));
      const bool mine = valid && cls == c;
      const double* S = Ct + kCtSelf + 64 * c;
      double v[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) v[m] = mine ? u0[m] : 0.0;
      block_product(S, v, acc);
      pending &= ~__ballot(mine);
    }
  }
  // the neighbours x-1, x+1, y-1, y+1, one ahead of its products
  auto neighbour = [&](int sn, double (&u)[8]) {
    const int off = sn == 0 ? -1 : (sn == 1 ? 1 : (sn == 2 ? -n : n));
    const bool in = valid && (sn == 0 ? ex > 0 : (sn == 1 ? ex < n - 1 : (sn == 2 ? ey > 0 : ey < n - 1)));
    load(id + 2 * (int64_t)off, in, u);
  };
  double un[4][8];
#pragma unroll
  for (int sn = 0; sn < 4; ++sn) neighbour(sn, un[sn]);
#pragma unroll
  for (int sn = 0; sn < 4; ++sn) block_product(Ct + kCtNbr + 64 * sn, un[sn], acc);
  // mass part: the diagonal component of this row (row k, component k) and the
  // other one; wv[r]: component r / 4, corner r % 4
  double wv[8];
  {
    double ud[4], uo[4], d[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      ud[m] = k ? u0[4 + m] : u0[m];
      uo[m] = k ? u0[m] : u0[4 + m];
      const double other = pair_swap(ud[m]);
      d[m] = k ? other - ud[m] : ud[m] - other;   // u11 - u22
    }
    const double* M = Ct + kCtMass;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double md = 0.5 * (M[4 * j] * d[0] + M[4 * j + 1] * d[1] + M[4 * j + 2] * d[2] + M[4 * j + 3] * d[3]);
      if (k) md = -md;
      const double mo = M[4 * j] * uo[0] + M[4 * j + 1] * uo[1] + M[4 * j + 2] * uo[2] + M[4 * j + 3] * uo[3];
      wv[j] = inv_nu * (k ? mo : md) + dt * acc[j];
      wv[4 + j] = inv_nu * (k ? md : mo) + dt * acc[4 + j];
    }
  }
  double dot = 0.0;
  if (MODE == kAstarResidual && valid) {
    double bv[8];
    ld4_any(b + 8 * (int64_t)id, bv);
    ld4_any(b + 8 * (int64_t)id + 4, bv + 4);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      wv[r] = bv[r] - wv[r];
      dot += wv[r] * wv[r];
    }
  }
  if (valid) {
    if (w) {
      st4_any(w + 8 * (int64_t)id, wv);
      st4_any(w + 8 * (int64_t)id + 4, wv + 4);
    }
    if (MODE == kAstarDir || MODE == kAstarFirst) {
      st4_any(p_new + 8 * (int64_t)id, u0);
      st4_any(p_new + 8 * (int64_t)id + 4, u0 + 4);
    }
  }
  if (s) {   // s = Z^T w: w11 of the even lane, w22 of the odd one
    double sv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) sv[j] = (wv[j] + pair_swap(wv[4 + j])) * kInvSqrt2;
    if (valid && !k) st4_any(s + 4 * (int64_t)e, sv);
  }
  if (MODE == kAstarResidual) {
    const double t = block_sum(dot, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
  }
}

// Row r of A_div Z at square e: the table's neighbour blocks and the own one of
// the square's class times z of the square and its neighbours; az in LDS.
__device__ __forceinline__ double az_row(const double* az, int r, int e, int n,
                                         const double* __restrict__ z) {
  const int ex = e & (n - 1), ey = e / n;
  double zc[5][4];
#pragma unroll
  for (int sn = 0; sn < 5; ++sn) {
    const int off = sn == 1 ? -1 : (sn == 2 ? 1 : (sn == 3 ? -n : (sn == 4 ? n : 0)));
    const bool in = sn == 0 || (sn == 1 ? ex > 0 : (sn == 2 ? ex < n - 1 : (sn == 3 ? ey > 0 : ey < n - 1)));
#pragma unroll
    for (int m = 0; m < 4; ++m) zc[sn][m] = 0.0;
    if (in) ld4_any(z + 4 * ((int64_t)e + off), zc[sn]);
  }
  double acc = 0.0;
#pragma unroll
  for (int sn = 0; sn < 5; ++sn) {
    const double2* c = reinterpret_cast<const double2*>(
        az + (sn == 0 ? kAzSelf + 64 * square_class(ex, ey, n) : kAzNbr + 64 * (sn - 1))) + r;
    const double2 c0 = c[0], c1 = c[16];
    acc += c0.x * zc[sn][0] + c0.y * zc[sn][1] + c1.x * zc[sn][2] + c1.y * zc[sn][3];
  }
  return acc;
}

__device__ __forceinline__ void az_stage(const double* __restrict__ AZ, double* az) {
  for (int i = threadIdx.x; i < kAzLen / 2; i += kThreads)
    reinterpret_cast<double2*>(az)[i] = reinterpret_cast<const double2*>(AZ)[i];
  __syncthreads();
}

// q = w - c (A_div Z) z, partial (p, q); prologue: r = w - c AZ z -> q, p_out,
// partials (w, w), (r, r).  Thread (square, row), 16 squares per workgroup and
// trip; a workgroup takes a contiguous range of squares and keeps the table
// (6.5 KB) in LDS: in registers it left 16 wavefronts a compute unit, too few
// to hide the trips' loads (35 us at n = 512, 32 us so).  Bound by w, p and q:
// 108 MB at n = 512 (128 us with the blocks of every square read from memory).
template <bool PROLOGUE>
__global__ __launch_bounds__(kThreads) void k_deflate(
    const double* __restrict__ AZ, int n, double c, const double* __restrict__ z,
    const double* __restrict__ w, const double* __restrict__ p, double* __restrict__ q,
    double* __restrict__ p_out, double* __restrict__ part, Slots sl) {
  __shared__ __align__(16) double az[kAzLen];
  __shared__ double lds[4];
  const int slot = slot_id(sl);
  z += slot * sl.sstride;
  w += slot * sl.tstride;
  if (p) p += slot * sl.tstride;
  q += slot * sl.tstride;
  if (p_out) p_out += slot * sl.tstride;
  part += slot * kSlotPart;
  const int ne = n * n, r = threadIdx.x & 15;
  const int groups = (ne + 15) >> 4, per = (groups + gridDim.x - 1) / gridDim.x;
  const int g0 = mg::xcd_band(blockIdx.x, gridDim.x) * per;
  const int g1 = g0 + per < groups ? g0 + per : groups;
  az_stage(AZ, az);
  double d0 = 0.0, d1 = 0.0;
#pragma unroll 2
  for (int g = g0; g < g1; ++g) {
    const int e = (g << 4) + (threadIdx.x >> 4);   // ne is a multiple of 16
    const int64_t i = 16 * (int64_t)e + r;
    const double wv = w[i];
    const double pv = PROLOGUE ? 0.0 : p[i];
    const double qv = wv - c * az_row(az, r, e, n, z);
    q[i] = qv;
    if (PROLOGUE) {
      p_out[i] = qv;
      d0 += wv * wv;
      d1 += qv * qv;
    } else {
      d0 += pv * qv;
    }
  }
  const double t0 = block_sum(d0, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t0;
  if (PROLOGUE) {
    const double t1 = block_sum(d1, lds);
    if (threadIdx.x == 0) part[kPartStride + blockIdx.x] = t1;
  }
}

__global__ __launch_bounds__(kThreads) void k_adivz(const double* __restrict__ AZ, int n,
                                                    const double* __restrict__ y,
                                                    double* __restrict__ out) {
  __shared__ __align__(16) double az[kAzLen];
  const int e = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int r = threadIdx.x & 15;
  az_stage(AZ, az);
  if (e >= n * n) return;
  out[16 * (int64_t)e + r] = az_row(az, r, e, n, y);
}

// x += alpha p; r -= alpha q; partial (r, r) [flexible: (r,q), (p,r)]
template <bool FLEX>
__global__ __launch_bounds__(kThreads) void k_cg_update(int64_t n, const Scalars* __restrict__ sc,
                                                        const double* __restrict__ p,
                                                        const double* __restrict__ q,
                                                        double* __restrict__ x,
                                                        double* __restrict__ r,
                                                        double* __restrict__ part, Slots sl) {
  __shared__ double lds[4];
  const int slot = slot_id(sl);
  p += slot * sl.tstride;
  q += slot * sl.tstride;
  x += slot * sl.tstride;
  r += slot * sl.tstride;
  sc += slot;
  part += slot * kSlotPart;
  const double alpha = sc->alpha;
  double rr = 0.0, rq = 0.0, pr = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    const double pi = p[i], qi = q[i];
    x[i] = x[i] + alpha * pi;
    const double ri = r[i] - alpha * qi;
    r[i] = ri;
    rr += ri * ri;
    if (FLEX) {
      rq += ri * qi;
      pr += pi * ri;
    }
  }
  const double t0 = block_sum(rr, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t0;
  if (FLEX) {
    const double t1 = block_sum(rq, lds);
    if (threadIdx.x == 0) part[kPartStride + blockIdx.x] = t1;
    const double t2 = block_sum(pr, lds);
    if (threadIdx.x == 0) part[2 * kPartStride + blockIdx.x] = t2;
  }
}

__global__ __launch_bounds__(kThreads) void k_axpy_dot(int64_t n, double a,
                                                       const double* __restrict__ q,
                                                       double* __restrict__ r,
                                                       double* __restrict__ part) {
  __shared__ double lds[4];
  double rr = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    const double ri = r[i] + a * q[i];
    r[i] = ri;
    rr += ri * ri;
  }
  const double t = block_sum(rr, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// One workgroup of 16 wavefronts: the partials of a launch are a few loads per
// thread, then a shuffle tree and one pass over the wavefront sums (fixed order).
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void k_reduce(const double* __restrict__ part, int nb,
                                                     int op, Scalars* __restrict__ sc, Slots sl,
                                                     double aux, int iaux) {
  __shared__ double sm[kReduceThreads / 64];
  const int slot = slot_id(sl);
  part += slot * kSlotPart;
  sc += slot;
  if (op == kRedInnerR2 && sc->inner_done) return;   // the partials were not recomputed
  const int nslot = op == kRedB2Rho ? 2 : (op == kRedFcgBeta ? 3 : 1);
  double sums[3] = {0.0, 0.0, 0.0};
  for (int slot = 0; slot < nslot; ++slot) {
    double v = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < nb; i += kReduceThreads) v += part[slot * kPartStride + i];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int i = 0; i < kReduceThreads / 64; ++i) t += sm[i];
      sums[slot] = t;
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  switch (op) {
    case kRedB2Rho:
      sc->b2 = sums[0];
      sc->rho = sums[1];
      sc->dr = sums[1];
      break;
    case kRedAlpha:
    case kRedFcgAlpha: {
      const double pq = sums[0];
      sc->pq = pq;
      if (!(pq > 0.0) || !isfinite(pq)) {
        sc->breakdown = 1;
        sc->alpha = 0.0;
      } else {
        sc->alpha = (op == kRedAlpha ? sc->rho : sc->dr) / pq;
      }
      break;
    }
    case kRedBeta:
      sc->beta = sc->rho > 0.0 ? sums[0] / sc->rho : 0.0;
      sc->rho = sums[0];
      sc->dr = sums[0];
      break;
    case kRedFcgBeta: {
      const double beta = sc->pq > 0.0 ? -sums[1] / sc->pq : 0.0;
      sc->rho = sums[0];
      sc->beta = beta;
      sc->dr = sums[0] + beta * sums[2];
      break;
    }
    case kRedS2:
      sc->s2 = sums[0];
      sc->r2 = sums[0];
      break;
    case kRedInnerS2:
      sc->s2 = sums[0];
      sc->r2 = sums[0];
      sc->inner_lim2 = aux * sums[0];
      sc->inner_cycles = 0;
      sc->inner_done = !(sums[0] > aux * sums[0]) || iaux <= 0;
      break;
    case kRedInnerR2:
      sc->r2 = sums[0];
      sc->inner_cycles += 1;
      sc->inner_done = !(sums[0] > sc->inner_lim2) || sc->inner_cycles >= iaux;
      break;
    case kRedR2:
      sc->r2 = sums[0];
      break;
    case kRedRes:
      sc->res2 = sums[0];
      break;
    case kRedRho:
      sc->rho = sums[0];
      sc->dr = sums[0];
      break;
    case kRedDr:
      sc->dr = sums[0];
      break;
  }
}

// Partial (r, q_k) for the k-th window direction (blockIdx.y = k).
__global__ __launch_bounds__(kThreads) void k_fcg_dot(int64_t n, const double* __restrict__ r,
                                                      const double* const* __restrict__ qptr,
                                                      int first, int R, double* __restrict__ part) {
  __shared__ double lds[4];
  const int k = blockIdx.y;
  const double* q = qptr[(first + k) % R];
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads)
    acc += r[i] * q[i];
  const double t = block_sum(acc, lds);
  if (threadIdx.x == 0) part[(int64_t)k * gridDim.x + blockIdx.x] = t;
}

// coef[k] = -(sum of the k-th partials, in block order) / dq_k (dq == nullptr: -sum).
__global__ __launch_bounds__(kThreads) void k_fcg_coef(const double* __restrict__ part, int nb,
                                                       const double* __restrict__ dq, int first,
                                                       int R, double* __restrict__ coef) {
  __shared__ double lds[4];
  const int k = blockIdx.x;
  double acc = 0.0;
  for (int b = threadIdx.x; b < nb; b += kThreads) acc += part[(int64_t)k * nb + b];
  const double t = block_sum(acc, lds);
  if (threadIdx.x == 0) coef[k] = dq ? -t / dq[(first + k) % R] : -t;
}

// d may alias r (in-place Gram-Schmidt update): element i is read before it is
// written by the same thread.
__global__ __launch_bounds__(kThreads) void k_fcg_direction(
    int64_t n, const double* r, const double* rdot, const double* const* __restrict__ dptr, int first,
    int m, int R, const double* __restrict__ coef, double* d, double* __restrict__ part) {
  __shared__ double lds[4];
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    const double ri = r[i];
    double di = ri;
    for (int k = 0; k < m; ++k) di += coef[k] * dptr[(first + k) % R][i];
    d[i] = di;
    acc += di * (rdot ? rdot[i] : ri);
  }
  const double t = block_sum(acc, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ __launch_bounds__(kThreads) void k_zt(int ne, const double* __restrict__ w,
                                                 double* __restrict__ s, Slots sl) {
  const int slot = slot_id(sl);
  w += slot * sl.tstride;
  s += slot * sl.sstride;
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= 4 * (int64_t)ne) return;
  const int64_t e = i >> 2, j = i & 3;
  s[i] = (w[16 * e + j] + w[16 * e + 12 + j]) * kInvSqrt2;
}

__global__ __launch_bounds__(kThreads) void k_z(int ne, const double* __restrict__ y, double c,
                                                double* __restrict__ v) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= 16 * (int64_t)ne) return;
  const int64_t e = i >> 4, cc = (i >> 2) & 3, j = i & 3;
  v[i] = (cc == 0 || cc == 3) ? (c * y[4 * e + j]) * kInvSqrt2 : 0.0;
}

// x = (xh - Z (c zt)) + Z (c zb)  (eq. (x_defl) with pi(b) reused)
__global__ __launch_bounds__(kThreads) void k_reconstruct(int ne, const double* __restrict__ xh,
                                                          const double* __restrict__ zt,
                                                          const double* __restrict__ zb,
                                                          const Scalars* __restrict__ sc,
                                                          double* __restrict__ x, Slots sl) {
  const int slot = slot_id(sl);
  xh += slot * sl.tstride;
  zt += slot * sl.sstride;
  zb += slot * sl.sstride;
  x += slot * sl.tstride;
  const double c = 2.0 / sc[slot].dt;
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= 16 * (int64_t)ne) return;
  const int64_t e = i >> 4, cc = (i >> 2) & 3, j = i & 3;
  double v = xh[i];
  if (cc == 0 || cc == 3) {
    v = v - (c * zt[4 * e + j]) * kInvSqrt2;
    v = v + (c * zb[4 * e + j]) * kInvSqrt2;
  }
  x[i] = v;
}

// BDF2 right-hand side and warm start: f = (1/nu) (C (x) M_1)(4/3 s1 - 1/3 s2)
// + c F, x0 = 2 s1 - s2; thread (square, row).
__global__ __launch_bounds__(kThreads) void k_bdf2_rhs(int ne, const double* __restrict__ Ct,
                                                       double inv_nu, const double* __restrict__ s1,
                                                       const double* __restrict__ s2,
                                                       const double* __restrict__ F, double c,
                                                       double* __restrict__ f,
                                                       double* __restrict__ x0) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i >= 16 * (int64_t)ne) return;
  const int64_t e = i >> 4;
  const int r = int(i & 15), cc = r >> 2, j = r & 3;
  double u[16];
#pragma unroll
  for (int k = 0; k < 16; ++k)
    u[k] = 4.0 / 3.0 * s1[16 * e + k] - 1.0 / 3.0 * s2[16 * e + k];
  double m[4];
  ld4_any(Ct + kCtMass + 4 * j, m);
  double mu;
  if (cc == 0 || cc == 3) {
    mu = 0.5 * (m[0] * (u[0] - u[12]) + m[1] * (u[1] - u[13]) + m[2] * (u[2] - u[14]) +
                m[3] * (u[3] - u[15]));
    if (cc == 3) mu = -mu;
  } else {
    const int o = 4 * cc;
    mu = m[0] * u[o] + m[1] * u[o + 1] + m[2] * u[o + 2] + m[3] * u[o + 3];
  }
  f[i] = inv_nu * mu + c * F[i];
  x0[i] = 2.0 * s1[i] - s2[i];
}

__global__ __launch_bounds__(kThreads) void k_scale(int64_t n, double c,
                                                    const double* __restrict__ in,
                                                    double* __restrict__ out) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i < n) out[i] = c * in[i];
}

// ============================================================ inner refinement
// r = s - L64 z (first: r = s) in FP64, fJ = (T) r, partial ||r||^2.
// Thread per square, one wavefront per workgroup, the operator rows from the class
// table in scalar registers: bound by bytes (20 MB at n = 512, FP32 levels: 4 us) and
// the latency of one round of loads, 13.7 -> 10.2 us with a thread per row reading
// the table and the stencil per row.
template <typename T, bool FIRST>
__global__ __launch_bounds__(64) void k_refine_residual(
    const double* __restrict__ Lc, int n, int ne, const double* __restrict__ s,
    const double* __restrict__ z, T* __restrict__ fJ, double* __restrict__ part, Slots sl,
    const Scalars* __restrict__ guard) {
  if (guard && guard->inner_done) return;
  const int slot = slot_id(sl);
  s += slot * sl.sstride;
  if (z) z += slot * sl.sstride;
  fJ += slot * sl.lstride;
  part += slot * kSlotPart;
  const int groups = (ne + 63) >> 6;
  double nrm = 0.0;
  for (int g = blockIdx.x; g < groups; g += gridDim.x) {
    const int e = (g << 6) + threadIdx.x;
    if (e >= ne) continue;
    double r[4];
    ld4_any(s + 4 * (int64_t)e, r);
    if (!FIRST) {                // blocks of the square's class, neighbours from (ex, ey)
      const int ex = e % n, ey = e / n;
      double zq[5][4], acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int sn = 0; sn < 5; ++sn) {
        const int dx = sn == 1 ? -1 : (sn == 2 ? 1 : 0), dy = sn == 3 ? -1 : (sn == 4 ? 1 : 0);
        zq[sn][0] = zq[sn][1] = zq[sn][2] = zq[sn][3] = 0.0;
        if (ex + dx >= 0 && ex + dx < n && ey + dy >= 0 && ey + dy < n)
          ld4_any(z + 4 * ((int64_t)e + dx + (int64_t)dy * n), zq[sn]);
      }
      mg::class_rows(Lc, square_class(ex, ey, n), zq, acc);
#pragma unroll
      for (int a = 0; a < 4; ++a) r[a] -= acc[a];
    }
    const T o[4] = {static_cast<T>(r[0]), static_cast<T>(r[1]), static_cast<T>(r[2]), static_cast<T>(r[3])};
    st4_any(fJ + e * sl.lsq, o);
    nrm += (r[0] * r[0] + r[1] * r[1]) + (r[2] * r[2] + r[3] * r[3]);
  }
  for (int o = 32; o > 0; o >>= 1) nrm += __shfl_xor(nrm, o);
  if (threadIdx.x == 0) part[blockIdx.x] = nrm;
}

// ============================================================ multigrid levels
// out = L z (RES = false) or out = f - L z (RES = true); thread (square, row).
template <typename T, bool RES>
__global__ __launch_bounds__(kThreads) void k_lap(const T* __restrict__ L,
                                                  const int32_t* __restrict__ cols, int ne,
                                                  const T* __restrict__ f, const T* __restrict__ z,
                                                  T* __restrict__ out) {
  const int e = blockIdx.x * 64 + (threadIdx.x >> 2);
  const int a = threadIdx.x & 3;
  if (e >= ne) return;
  T acc = T(0);
#pragma unroll
  for (int slot = 0; slot < 5; ++slot) {
    const int col = cols[slot * ne + e];
    if (col < 0) continue;
    T l[4], zc[4];
    ld4_any(L + (((int64_t)slot * ne + e) * 4 + a) * 4, l);
    ld4_any(z + 4 * (int64_t)col, zc);
    acc += l[0] * zc[0] + l[1] * zc[1] + l[2] * zc[2] + l[3] * zc[3];
  }
  const int64_t i = 4 * (int64_t)e + a;
  out[i] = RES ? f[i] - acc : acc;
}

// Coefficient of coarse corner A at fine corner a of child ch: the coarse
// bilinear function at ((ch_x + a_x)/2, (ch_y + a_y)/2); values in
// {0, 1/4, 1/2, 1}, exact in any precision.
template <typename T>
__device__ inline T pcoef(int ch, int a, int A) {
  const int px = (ch & 1) + (a & 1), py = (ch >> 1) + (a >> 1);   // position in halves
  const int wx = (A & 1) ? px : 2 - px, wy = (A >> 1) ? py : 2 - py;
  return T(wx * wy) * T(0.25);
}

// rc = P^T r; thread per coarse dof (E, A)
template <typename T>
__global__ __launch_bounds__(kThreads) void k_restrict(int nc, const T* __restrict__ r,
                                                       T* __restrict__ rc) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  const int64_t nec = (int64_t)nc * nc;
  if (i >= 4 * nec) return;
  const int64_t E = i >> 2;
  const int A = int(i & 3);
  const int EX = int(E % nc), EY = int(E / nc);
  const int nf = 2 * nc;
  T acc = T(0);
#pragma unroll
  for (int ch = 0; ch < 4; ++ch) {
    const int64_t e = (int64_t)(2 * EY + (ch >> 1)) * nf + 2 * EX + (ch & 1);
    T v[4];
    ld4_any(r + 4 * e, v);
#pragma unroll
    for (int a = 0; a < 4; ++a) acc += pcoef<T>(ch, a, A) * v[a];
  }
  rc[i] = acc;
}

// z += P ec; thread per fine dof (e, a)
template <typename T>
__global__ __launch_bounds__(kThreads) void k_prolong(int nc, const T* __restrict__ ec,
                                                      T* __restrict__ z) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  const int nf = 2 * nc;
  if (i >= 4 * (int64_t)nf * nf) return;
  const int64_t e = i >> 2;
  const int a = int(i & 3);
  const int ex = int(e % nf), ey = int(e / nf);
  const int ch = (ex & 1) + 2 * (ey & 1);
  const int64_t E = (int64_t)(ey >> 1) * nc + (ex >> 1);
  T v[4];
  ld4_any(ec + 4 * E, v);
  T acc = T(0);
#pragma unroll
  for (int A = 0; A < 4; ++A) acc += pcoef<T>(ch, a, A) * v[A];
  z[i] = z[i] + acc;
}

// z = L_1^{-1} f with the FP64 inverse; one wavefront per row.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_coarse(const double* __restrict__ inv,
                                                     const T* __restrict__ f, T* __restrict__ z) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= 1024) return;
  const double* ir = inv + (int64_t)row * 1024;
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int j = lane + 64 * m;
    acc += ir[j] * static_cast<double>(f[j]);
  }
  acc = wave_sum(acc);
  if (lane == 0) z[row] = static_cast<T>(acc);
}

// z = A f, A dense FP64: one wavefront per row, lanes over pairs of columns, a
// fixed shuffle sum.  Bound by the matrix (134 MB at m = 4096).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_fold(int m, const double* __restrict__ A,
                                                   const T* __restrict__ f, T* __restrict__ z) {
  const int i = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (i >= m) return;   // whole wavefronts
  const double2* row = reinterpret_cast<const double2*>(A + (int64_t)i * m);
  double acc = 0.0;
#pragma unroll 8
  for (int j = threadIdx.x & 63; j < m / 2; j += 64) {
    const double2 a = row[j];
    acc += a.x * static_cast<double>(f[2 * j]) + a.y * static_cast<double>(f[2 * j + 1]);
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) z[i] = static_cast<T>(acc);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_fill(int64_t n, T v, T* __restrict__ x) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i < n) x[i] = v;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_copy(int64_t n, const T* __restrict__ x,
                                                   T* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (i < n) y[i] = x[i];
}

}  // namespace

// ============================================================ launchers
hipError_t launch_astar(int mode, const double* Ct, int n, const double* x, const double* p_old,
                        const double* b, const Scalars* sc, double* p_new, double* w, double* s,
                        double* part, hipStream_t st, const Slots& sl, int count, hipEvent_t ev0,
                        hipEvent_t ev1) {
  if (n < 16 || (n & (n - 1))) return hipErrorInvalidValue;   // squares of a row by masking
  const dim3 grid(astar_blocks(n * n), count);
  // timed launches record their events in the dispatch packet itself
#define DCG_ASTAR(M)                                                                            \
  hipExtLaunchKernelGGL(k_astar<M>, grid, dim3(kThreads), 0, st, ev0, ev1, 0, Ct, n, x, p_old, b, \
                        sc, p_new, w, s, part, sl)
  switch (mode) {
    case kAstarPlain: DCG_ASTAR(kAstarPlain); break;
    case kAstarDir: DCG_ASTAR(kAstarDir); break;
    case kAstarFirst: DCG_ASTAR(kAstarFirst); break;
    case kAstarResidual: DCG_ASTAR(kAstarResidual); break;
    default: return hipErrorInvalidValue;
  }
#undef DCG_ASTAR
  return hipGetLastError();
}

// one thread per square and stress row; n <= 2048 keeps it under kPartStride
int astar_blocks(int ne) { return (2 * ne + kThreads - 1) / kThreads; }
int deflate_blocks(int ne) { return grid_for(ne, 16, 2048); }

hipError_t launch_deflate(bool prologue, const double* AZ, int n, double c, const double* z,
                          const double* w, const double* p, double* q, double* p_out, double* part,
                          hipStream_t st, const Slots& sl, int count) {
  if (n < 16 || (n & (n - 1))) return hipErrorInvalidValue;
  const dim3 grid(deflate_blocks(n * n), count);
  if (prologue)
    k_deflate<true><<<grid, kThreads, 0, st>>>(AZ, n, c, z, w, p, q, p_out, part, sl);
  else
    k_deflate<false><<<grid, kThreads, 0, st>>>(AZ, n, c, z, w, p, q, p_out, part, sl);
  return hipGetLastError();
}

hipError_t launch_adivz(const double* AZ, int n, const double* y, double* out, hipStream_t st) {
  if (n < 16 || (n & (n - 1))) return hipErrorInvalidValue;
  k_adivz<<<grid_for(n * n, 16, 1 << 30), kThreads, 0, st>>>(AZ, n, y, out);
  return hipGetLastError();
}

hipError_t launch_cg_update(bool flexible, int64_t nvec, const Scalars* sc, const double* p,
                            const double* q, double* x, double* r, double* part, int* nblocks,
                            hipStream_t st, const Slots& sl, int count) {
  const int gx = grid_for(nvec, kThreads * 4, 8192);
  *nblocks = gx;
  const dim3 grid(gx, count);
  if (flexible)
    k_cg_update<true><<<grid, kThreads, 0, st>>>(nvec, sc, p, q, x, r, part, sl);
  else
    k_cg_update<false><<<grid, kThreads, 0, st>>>(nvec, sc, p, q, x, r, part, sl);
  return hipGetLastError();
}

int fcg_coef_blocks(int64_t n) { return grid_for(n, kThreads * 8, 128); }

hipError_t launch_fcg_coef(int64_t n, const double* r, const double* const* qptr, const double* dq,
                           int first, int m, int R, double* part, double* coef, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  const int nb = fcg_coef_blocks(n);
  k_fcg_dot<<<dim3(nb, m), kThreads, 0, st>>>(n, r, qptr, first, R, part);
  k_fcg_coef<<<m, kThreads, 0, st>>>(part, nb, dq, first, R, coef);
  return hipGetLastError();
}

hipError_t launch_fcg_direction(int64_t n, const double* r, const double* rdot, const double* const* dptr, int first,
                                int m, int R, const double* coef, double* d, double* part,
                                int* nblocks, hipStream_t st) {
  const int grid = grid_for(n, kThreads * 4, 8192);
  *nblocks = grid;
  k_fcg_direction<<<grid, kThreads, 0, st>>>(n, r, rdot, dptr, first, m, R, coef, d, part);
  return hipGetLastError();
}

hipError_t launch_axpy_dot(int64_t nvec, double a, const double* q, double* r, double* part,
                           int* nblocks, hipStream_t st) {
  const int grid = grid_for(nvec, kThreads * 4, 8192);
  *nblocks = grid;
  k_axpy_dot<<<grid, kThreads, 0, st>>>(nvec, a, q, r, part);
  return hipGetLastError();
}

hipError_t launch_reduce(const double* part, int nblocks, int op, Scalars* sc, hipStream_t st,
                         const Slots& sl, int count, double aux, int iaux) {
  k_reduce<<<dim3(1, count), kReduceThreads, 0, st>>>(part, nblocks, op, sc, sl, aux, iaux);
  return hipGetLastError();
}

hipError_t launch_zt(int ne, const double* w, double* s, hipStream_t st, const Slots& sl, int count) {
  k_zt<<<dim3(grid_for(4 * (int64_t)ne, kThreads, 1 << 30), count), kThreads, 0, st>>>(ne, w, s, sl);
  return hipGetLastError();
}

hipError_t launch_z(int ne, const double* y, double scale, double* v, hipStream_t st) {
  k_z<<<grid_for(16 * (int64_t)ne, kThreads, 1 << 30), kThreads, 0, st>>>(ne, y, scale, v);
  return hipGetLastError();
}

hipError_t launch_reconstruct(int ne, const double* xh, const double* zt, const double* zb,
                              const Scalars* sc, double* x, hipStream_t st, const Slots& sl,
                              int count) {
  k_reconstruct<<<dim3(grid_for(16 * (int64_t)ne, kThreads, 1 << 30), count), kThreads, 0, st>>>(
      ne, xh, zt, zb, sc, x, sl);
  return hipGetLastError();
}

hipError_t launch_bdf2_rhs(int ne, const double* Ct, double inv_nu, const double* s1,
                           const double* s2, const double* F, double c, double* f, double* x0,
                           hipStream_t st) {
  k_bdf2_rhs<<<grid_for(16 * (int64_t)ne, kThreads, 1 << 30), kThreads, 0, st>>>(ne, Ct, inv_nu, s1, s2,
                                                                                F, c, f, x0);
  return hipGetLastError();
}

hipError_t launch_scale(int64_t n, double c, const double* in, double* out, hipStream_t st) {
  k_scale<<<grid_for(n, kThreads, 1 << 30), kThreads, 0, st>>>(n, c, in, out);
  return hipGetLastError();
}

int refine_blocks(int ne) { return grid_for(ne, 64, kPartStride); }

template <typename T>
hipError_t launch_refine_residual(bool first, const double* Lc64, int n, int ne, const double* s,
                                  const double* z, T* fJ, double* part, hipStream_t st,
                                  const Slots& sl, int count, const Scalars* guard) {
  if (!Lc64 || n < 3 || int64_t(n) * n != ne) return hipErrorInvalidValue;
  const dim3 grid(refine_blocks(ne), count);
  if (first)
    k_refine_residual<T, true><<<grid, 64, 0, st>>>(Lc64, n, ne, s, z, fJ, part, sl, guard);
  else
    k_refine_residual<T, false><<<grid, 64, 0, st>>>(Lc64, n, ne, s, z, fJ, part, sl, guard);
  return hipGetLastError();
}


template <typename T>
hipError_t launch_lap(bool residual, const T* L, const int32_t* cols, int ne, const T* f, const T* z,
                      T* out, hipStream_t st) {
  const int grid = grid_for(ne, 64, 1 << 30);
  if (residual)
    k_lap<T, true><<<grid, kThreads, 0, st>>>(L, cols, ne, f, z, out);
  else
    k_lap<T, false><<<grid, kThreads, 0, st>>>(L, cols, ne, f, z, out);
  return hipGetLastError();
}



template <typename T>
hipError_t launch_restrict(int nc, const T* r, T* rc, hipStream_t st) {
  k_restrict<T><<<grid_for(4 * (int64_t)nc * nc, kThreads, 1 << 30), kThreads, 0, st>>>(nc, r, rc);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_prolong(int nc, const T* ec, T* z, hipStream_t st) {
  k_prolong<T><<<grid_for(16 * (int64_t)nc * nc, kThreads, 1 << 30), kThreads, 0, st>>>(nc, ec, z);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_coarse(const double* inv, const T* f, T* z, hipStream_t st) {
  k_coarse<T><<<256, kThreads, 0, st>>>(inv, f, z);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fold(int m, const double* A, const T* f, T* z, hipStream_t st) {
  if (m <= 0 || m % 16) return hipErrorInvalidValue;
  k_fold<T><<<m / (kThreads / 64), kThreads, 0, st>>>(m, A, f, z);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fill(int64_t n, T v, T* x, hipStream_t st) {
  k_fill<T><<<grid_for(n, kThreads, 1 << 30), kThreads, 0, st>>>(n, v, x);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_copy(int64_t n, const T* x, T* y, hipStream_t st) {
  k_copy<T><<<grid_for(n, kThreads, 1 << 30), kThreads, 0, st>>>(n, x, y);
  return hipGetLastError();
}

#define DCG_INSTANTIATE(T)                                                                      \
  template hipError_t launch_refine_residual<T>(bool, const double*, int, int, const double*,  \
                                                const double*, T*, double*, hipStream_t,       \
                                                const Slots&, int, const Scalars*);            \
  template hipError_t launch_lap<T>(bool, const T*, const int32_t*, int, const T*, const T*, T*, \
                                    hipStream_t);                                              \
  template hipError_t launch_restrict<T>(int, const T*, T*, hipStream_t);                      \
  template hipError_t launch_prolong<T>(int, const T*, T*, hipStream_t);                       \
  template hipError_t launch_coarse<T>(const double*, const T*, T*, hipStream_t);              \
  template hipError_t launch_fold<T>(int, const double*, const T*, T*, hipStream_t);           \
  template hipError_t launch_fill<T>(int64_t, T, T*, hipStream_t);                             \
  template hipError_t launch_copy<T>(int64_t, const T*, T*, hipStream_t);

DCG_INSTANTIATE(float)
DCG_INSTANTIATE(double)

}  // namespace dcg

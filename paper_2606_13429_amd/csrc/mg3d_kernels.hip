// Kernels of the three-dimensional multigrid inner solve (Section 4.2, the 3D
// case; layouts in mg3d.hpp).  Level vectors hold 8 FP64 values per cube.
// The residual and the RAS step run as MFMA products over tasks of 16 cubes of
// a class on large levels and split every output over a few lanes on small
// ones; the transfers run one thread per (cube, row).  The class tables (operator
// 27 x 7 blocks, RAS updates 343 x 8 x 200) are shared by every cube of a
// class and stay in the caches.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "dcg3d.hpp"
#include "mg3d.hpp"
#include "mg_common.hpp"

namespace dcg3 {

namespace {

using dcg::mg::ld2_any;   // the caller's vectors
using dcg::mg::st2_any;

constexpr int kThreads = 256;
constexpr int kCubesPerBlock = kThreads / 8;

__device__ __forceinline__ int op_axis(int x, int n) { return x == 0 ? 0 : (x == n - 1 ? 2 : 1); }
__device__ __forceinline__ int ras_axis(int x, int n) {
  return x < 3 ? x : (n - 1 - x < 3 ? 6 - (n - 1 - x) : 3);
}

__device__ __forceinline__ bool stopped(const int32_t* guard) { return guard && *guard == 0; }

// Sum over the workgroup in a fixed order; valid in thread 0.
__device__ double block_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  return sh[0];
}

// The diamond (|dx| + |dy| + |dz| <= 2) as cube offsets, in the order of
// diamond_offsets().
struct DiamondOff {
  int d[kDiamond][3];
  constexpr DiamondOff() : d() {
    int k = 0;
    for (int dz = -2; dz <= 2; ++dz)
      for (int dy = -2; dy <= 2; ++dy)
        for (int dx = -2; dx <= 2; ++dx) {
          const int a = (dx < 0 ? -dx : dx) + (dy < 0 ? -dy : dy) + (dz < 0 ? -dz : dz);
          if (a <= 2) {
            d[k][0] = dx;
            d[k][1] = dy;
            d[k][2] = dz;
            ++k;
          }
        }
  }
};

// ---- residual and RAS step on large levels (n_k > kSplitMaxN): one wavefront
// per task of 16 cubes of one class, the class's rows times the cubes' gathered
// inputs as FP64 MFMA products.  Lane l supplies input values 2 q, 2 q + 1 (q =
// l / 16) of the neighbour cubes of cube l % 16 -- one 16-byte load and two
// 16 x 16 x 4 steps per neighbour -- and the table entry of row 2 (m & 3) +
// (m >> 2 & 1), m = l % 16, at the same column (rows 8..15 of the product repeat
// rows 0..7), and receives rows 2 q, 2 q + 1 of its cube.  Every operand comes
// from L1 / L2 with no LDS and no barrier; the class tables (12.8 KB) stay in L1
// for the tasks of the interior.  Bound by the load latency and the matrix rate (50
// steps of a RAS task are 1.3 us).  A task holds one class, so the 1/2 to 1/4 of
// a level that lies near the boundary costs what the interior does; bricks of
// 4 x 4 x 4 cubes in LDS, a table entry loaded per lane, took 28.8 us a RAS step
// and 13.0 us a residual at n = 32, the split kernels below 12.5 and 5.1 us at
// n = 16; tasks take 12.9 and 5.4 us, 5.2 and 3.8 us.
typedef double v4d __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4d mfma64(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int kInterior = 3 + 7 * 3 + 49 * 3;   // class at least 3 cubes from every side

struct Task {
  int q, row;        // lane group; table row of the lane
  int cls;           // RAS class
  int x, y, z, e;    // the lane's cube
  bool valid;
};

// Workgroups go round robin to the 8 XCDs: each takes a contiguous run of tasks,
// so that the cubes it reads share its L2 (remainder tasks keep their index).
__device__ __forceinline__ int xcd_index(int b, int G) {
  const int per = G >> 3;
  return b < 8 * per ? (b & 7) * per + (b >> 3) : b;
}

__device__ __forceinline__ Task load_task(int n, const int32_t* __restrict__ cubes,
                                          const int32_t* __restrict__ cls, int tasks) {
  Task t;
  const int lane = threadIdx.x, id = xcd_index(blockIdx.x, tasks);
  t.q = lane >> 4;
  t.row = 2 * (lane & 3) + ((lane >> 2) & 1);
  t.cls = cls[id];
  const int e = cubes[16 * id + (lane & 15)];
  t.valid = e >= 0;
  t.e = e >= 0 ? e : ~e;   // padding repeats a cube of the task
  t.x = t.e % n;
  t.y = (t.e / n) % n;
  t.z = t.e / (n * n);
  return t;
}

// Values 2 q, 2 q + 1 of the cube at offset (dx, dy, dz), zero outside the
// domain; IN: the task's class has every such cube inside (no tests, one
// base address).
template <bool IN>
__device__ __forceinline__ double2 task_input(const Task& t, int n, int dx, int dy, int dz,
                                              const double* __restrict__ v) {
  const double* own = v + 8 * (int64_t)t.e + 2 * t.q;
  const int64_t o = 8 * ((dz * n + dy) * n + dx);
  if (IN) return ld2_any(own + o);
  // the load is unconditional (from the cube itself outside the domain)
  const int x = t.x + dx, y = t.y + dy, z = t.z + dz;
  const bool in = x >= 0 && y >= 0 && z >= 0 && x < n && y < n && z < n;
  double2 r = ld2_any(own + (in ? o : 0));
  r.x = in ? r.x : 0.0;
  r.y = in ? r.y : 0.0;
  return r;
}

// The products of one task: residual terms L z (7 face slots) or the RAS update
// (25 diamond cubes); A points at the lane's table entries.
template <bool IN>
__device__ __forceinline__ void res_products(const Task& t, int n, const double* __restrict__ A,
                                             const double* __restrict__ z, v4d& a0, v4d& a1) {
  double2 v[kSlots];
#pragma unroll
  for (int s = 0; s < kSlots; ++s) {
    const int dx = s == 1 ? -1 : (s == 2 ? 1 : 0), dy = s == 3 ? -1 : (s == 4 ? 1 : 0),
              dz = s == 5 ? -1 : (s == 6 ? 1 : 0);
    v[s] = task_input<IN>(t, n, dx, dy, dz, z);
  }
#pragma unroll
  for (int s = 0; s < kSlots; ++s) {
    a0 = mfma64(A[64 * s], v[s].x, a0);
    a1 = mfma64(A[64 * s + 8], v[s].y, a1);
  }
}

template <bool IN>
__device__ __forceinline__ void ras_products(const Task& t, int n, const double* __restrict__ A,
                                             const double* __restrict__ r, v4d& a0, v4d& a1) {
  constexpr DiamondOff D;
  double2 v[kDiamond];
#pragma unroll
  for (int d = 0; d < kDiamond; ++d) v[d] = task_input<IN>(t, n, D.d[d][0], D.d[d][1], D.d[d][2], r);
#pragma unroll
  for (int d = 0; d < kDiamond; ++d) {
    a0 = mfma64(A[64 * d], v[d].x, a0);
    a1 = mfma64(A[64 * d + 8], v[d].y, a1);
  }
}

__global__ __launch_bounds__(64) void k_mg3_res(int n, int tasks, const int32_t* __restrict__ cubes,
                                                      const int32_t* __restrict__ tcls,
                                                      const double* __restrict__ opT,
                                                      const double* __restrict__ f,
                                                      const double* __restrict__ z,
                                                      double* __restrict__ r,
                                                      double* __restrict__ part,
                                                      const int32_t* __restrict__ guard) {
  if (stopped(guard)) return;
  const Task t = load_task(n, cubes, tcls, tasks);
  // operator class: 0 low side, 2 high side, 1 inside of the distance class
  const int p[3] = {t.cls % 7, (t.cls / 7) % 7, t.cls / 49};
  int oc = 0;
#pragma unroll
  for (int a = 2; a >= 0; --a) oc = 3 * oc + (p[a] == 0 ? 0 : (p[a] == 6 ? 2 : 1));
  // opT[cls][slot][b][row]
  const double* A = opT + (int64_t)oc * kSlots * 64 + 16 * t.q + t.row;
  v4d a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0;
  if (z) {
    if (t.cls == kInterior) res_products<true>(t, n, A, z, a0, a1);
    else res_products<false>(t, n, A, z, a0, a1);
  }
  double2 rv = make_double2(0.0, 0.0);
  if (t.valid) {
    if (f) rv = ld2_any(f + 8 * (int64_t)t.e + 2 * t.q);
    rv.x -= a0[0] + a1[0];
    rv.y -= a0[1] + a1[1];
    st2_any(r + 8 * (int64_t)t.e + 2 * t.q, rv.x, rv.y);
  }
  if (part) {   // the task's sum of r^2, fixed order
    double v = rv.x * rv.x + rv.y * rv.y;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    if (threadIdx.x == 0) part[blockIdx.x] = v;
  }
}

__global__ __launch_bounds__(64) void k_mg3_ras(int n, int tasks, const int32_t* __restrict__ cubes,
                                                      const int32_t* __restrict__ tcls,
                                                      const double* __restrict__ rasT,
                                                      const double* __restrict__ r,
                                                      double* __restrict__ z, int zero,
                                                      const int32_t* __restrict__ guard) {
  if (stopped(guard)) return;
  const Task t = load_task(n, cubes, tcls, tasks);
  // rasT[cls][column 200][row]
  const double* A = rasT + (int64_t)t.cls * 8 * kRasCols + 16 * t.q + t.row;
  double2 zv = make_double2(0.0, 0.0);
  if (t.valid && !zero) zv = ld2_any(z + 8 * (int64_t)t.e + 2 * t.q);
  v4d a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0;
  if (t.cls == kInterior) ras_products<true>(t, n, A, r, a0, a1);
  else ras_products<false>(t, n, A, r, a0, a1);
  if (t.valid) {
    zv.x += a0[0] + a1[0];
    zv.y += a0[1] + a1[1];
    st2_any(z + 8 * (int64_t)t.e + 2 * t.q, zv.x, zv.y);
  }
}

// ---- residual and RAS step on small levels (n_k <= kSplitMaxN): one lane
// per (cube, row, term group), so that every lane issues a single round of
// loads -- the table row segment and the neighbour's values, 64 bytes each
// -- and the groups are summed by a fixed shuffle tree.  These levels use
// the row-major tables.
// RAS: 32 lanes per output (lane d < 25 takes diamond cube d), 8 outputs per
// 256-thread workgroup.
__global__ __launch_bounds__(kThreads) void k_mg3_ras_split(int n, const double* __restrict__ ras,
                                                            const double* __restrict__ r,
                                                            double* __restrict__ z, int zero,
                                                            const int32_t* __restrict__ guard) {
  if (stopped(guard)) return;
  constexpr DiamondOff D;
  const int64_t ne = (int64_t)n * n * n;
  const int64_t out = (int64_t)blockIdx.x * (kThreads / 32) + (threadIdx.x >> 5);
  const int d = threadIdx.x & 31;
  const int64_t e = out >> 3;
  const int row = int(out & 7);
  double acc = 0.0;
  if (e < ne && d < kDiamond) {
    const int x = int(e % n), y = int((e / n) % n), zz = int(e / ((int64_t)n * n));
    const int qx = x + D.d[d][0], qy = y + D.d[d][1], qz = zz + D.d[d][2];
    if (qx >= 0 && qy >= 0 && qz >= 0 && qx < n && qy < n && qz < n) {
      const int cls = n < kRasClassMinN ? int(e) : ras_axis(x, n) + 7 * ras_axis(y, n) + 49 * ras_axis(zz, n);
      const double* K = ras + ((int64_t)cls * 8 + row) * kRasCols + 8 * d;
      const double* rn = r + 8 * (((int64_t)qz * n + qy) * n + qx);
#pragma unroll
      for (int b = 0; b < 8; ++b) acc += K[b] * rn[b];
    }
  }
#pragma unroll
  for (int m = 16; m > 0; m >>= 1) acc += __shfl_xor(acc, m, 32);
  if (d == 0 && e < ne) z[8 * e + row] = (zero ? 0.0 : z[8 * e + row]) + acc;
}

// Residual: 8 lanes per output (lane s < 7 takes face slot s), 32 outputs per
// 256-thread workgroup; with part, the workgroup's sum of r^2.
__global__ __launch_bounds__(kThreads) void k_mg3_res_split(int n, const double* __restrict__ op,
                                                            const double* __restrict__ f,
                                                            const double* __restrict__ z,
                                                            double* __restrict__ r,
                                                            double* __restrict__ part,
                                                            const int32_t* __restrict__ guard) {
  if (stopped(guard)) return;
  __shared__ double sh[kThreads / 64];
  const int64_t ne = (int64_t)n * n * n;
  const int64_t out = (int64_t)blockIdx.x * (kThreads / 8) + (threadIdx.x >> 3);
  const int s = threadIdx.x & 7;
  const int64_t e = out >> 3;
  const int row = int(out & 7);
  double acc = 0.0;
  if (e < ne && s < kSlots && z) {
    const int c[3] = {int(e % n), int((e / n) % n), int(e / ((int64_t)n * n))};
    const int ax = s == 0 ? 0 : (s - 1) >> 1;
    const int dir = s == 0 ? 0 : ((s & 1) ? -1 : 1);
    const int q = c[ax] + dir;
    if (q >= 0 && q < n) {
      const int cls = op_axis(c[0], n) + 3 * op_axis(c[1], n) + 9 * op_axis(c[2], n);
      const int64_t nb = e + dir * (ax == 0 ? 1 : (ax == 1 ? (int64_t)n : (int64_t)n * n));
      const double* row_p = op + ((cls * kSlots + s) * 8 + row) * 8;
      const double* zn = z + 8 * nb;
#pragma unroll
      for (int b = 0; b < 8; ++b) acc -= row_p[b] * zn[b];
    }
  }
#pragma unroll
  for (int m = 4; m > 0; m >>= 1) acc += __shfl_xor(acc, m, 8);
  double v = 0.0;
  if (s == 0 && e < ne) {
    acc += f ? f[8 * e + row] : 0.0;
    r[8 * e + row] = acc;
    v = acc * acc;
  }
  if (part) {   // the workgroup's sum of r^2, fixed order: lanes, then wavefronts
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      double sum = 0.0;
      for (int w = 0; w < kThreads / 64; ++w) sum += sh[w];
      part[blockIdx.x] = sum;
    }
  }
}

__device__ __forceinline__ double inject(int q, int i, int J) {
  double v = 1.0;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    const double t = 0.5 * (((q >> ax) & 1) + ((i >> ax) & 1));
    v *= ((J >> ax) & 1) ? t : 1.0 - t;
  }
  return v;
}

__global__ __launch_bounds__(kThreads) void k_mg3_restrict(int nf, const double* __restrict__ r,
                                                           double* __restrict__ fc,
                                                           const int32_t* __restrict__ guard) {
  if (stopped(guard)) return;
  const int nc = nf / 2;
  const int64_t nec = (int64_t)nc * nc * nc;
  const int64_t E = (int64_t)blockIdx.x * kCubesPerBlock + threadIdx.x / 8;
  const int J = threadIdx.x & 7;
  if (E >= nec) return;
  const int X = int(E % nc), Y = int((E / nc) % nc), Z = int(E / ((int64_t)nc * nc));
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int64_t c = ((int64_t)(2 * Z + (q >> 2)) * nf + 2 * Y + ((q >> 1) & 1)) * nf + 2 * X + (q & 1);
    const double* rc = r + 8 * c;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc += inject(q, i, J) * rc[i];
  }
  fc[8 * E + J] = acc;
}

__global__ __launch_bounds__(kThreads) void k_mg3_prolong(int nf, const double* __restrict__ zc,
                                                          double* __restrict__ z, int assign,
                                                          const int32_t* __restrict__ guard) {
  if (stopped(guard)) return;
  const int nc = nf / 2;
  const int64_t ne = (int64_t)nf * nf * nf;
  const int64_t e = (int64_t)blockIdx.x * kCubesPerBlock + threadIdx.x / 8;
  const int i = threadIdx.x & 7;
  if (e >= ne) return;
  const int x = int(e % nf), y = int((e / nf) % nf), zz = int(e / ((int64_t)nf * nf));
  const int q = (x & 1) | ((y & 1) << 1) | ((zz & 1) << 2);
  const double* zE = zc + 8 * (((int64_t)(zz >> 1) * nc + (y >> 1)) * nc + (x >> 1));
  double acc = 0.0;
#pragma unroll
  for (int J = 0; J < 8; ++J) acc += inject(q, i, J) * zE[J];
  z[8 * e + i] = assign ? acc : z[8 * e + i] + acc;
}

// z = A f, A dense m x m (m even): one wavefront per row, lanes over pairs of
// columns, a fixed shuffle sum.  Bound by the matrix (134 MB at m = 4096).
__global__ __launch_bounds__(kThreads) void k_mg3_dense(int m, const double* __restrict__ A,
                                                        const double* __restrict__ f,
                                                        double* __restrict__ z,
                                                        const int32_t* __restrict__ guard) {
  if (stopped(guard)) return;
  const int i = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (i >= m) return;   // whole wavefronts
  const double2* row = reinterpret_cast<const double2*>(A + (int64_t)i * m);
  double acc = 0.0;
#pragma unroll 8
  for (int j = threadIdx.x & 63; j < m / 2; j += 64) {
    const double2 a = row[j], b = ld2_any(f + 2 * j);
    acc += a.x * b.x + a.y * b.y;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);
  if ((threadIdx.x & 63) == 0) z[i] = acc;
}

// The residual and the RAS step of a small level on the m columns of a matrix Z at
// once (set-up; row-major tables): thread (cube, column), the table rows through
// scalar loads, the columns of a wavefront contiguous.  R = I - L Z (Z = NULL: R = I).
__global__ __launch_bounds__(64) void k_mg3_res_cols(int n, const double* __restrict__ op,
                                                     const double* __restrict__ Z,
                                                     double* __restrict__ R) {
  const int64_t m = 8 * (int64_t)n * n * n;
  const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int e = blockIdx.y, c[3] = {e % n, (e / n) % n, e / (n * n)};
  const int cls = op_axis(c[0], n) + 3 * op_axis(c[1], n) + 9 * op_axis(c[2], n);
  double acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 8 * (int64_t)e + i == j ? 1.0 : 0.0;
  for (int s = 0; Z && s < kSlots; ++s) {
    const int ax = s == 0 ? 0 : (s - 1) >> 1, dir = s == 0 ? 0 : ((s & 1) ? -1 : 1);
    const int q = (ax == 0 ? c[0] : (ax == 1 ? c[1] : c[2])) + dir;
    if (q < 0 || q >= n) continue;
    const int nb = e + dir * (ax == 0 ? 1 : (ax == 1 ? n : n * n));
    const double* B = op + (cls * kSlots + s) * 64;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const double v = Z[(8 * (int64_t)nb + b) * m + j];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] -= B[8 * i + b] * v;
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) R[(8 * (int64_t)e + i) * m + j] = acc[i];
}

// Z = (zero ? 0 : Z) + S R.
__global__ __launch_bounds__(64) void k_mg3_ras_cols(int n, const double* __restrict__ ras,
                                                     const double* __restrict__ R,
                                                     double* __restrict__ Z, int zero) {
  constexpr DiamondOff D;
  const int64_t m = 8 * (int64_t)n * n * n;
  const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int e = blockIdx.y, x = e % n, y = (e / n) % n, z = e / (n * n);
  const int cls = n < kRasClassMinN ? e : ras_axis(x, n) + 7 * ras_axis(y, n) + 49 * ras_axis(z, n);
  const double* K = ras + (int64_t)cls * 8 * kRasCols;
  double acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.0;
  for (int d = 0; d < kDiamond; ++d) {
    const int qx = x + D.d[d][0], qy = y + D.d[d][1], qz = z + D.d[d][2];
    if (qx < 0 || qy < 0 || qz < 0 || qx >= n || qy >= n || qz >= n) continue;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const double v = R[(8 * (((int64_t)qz * n + qy) * n + qx) + b) * m + j];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += K[kRasCols * i + 8 * d + b] * v;
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    double* p = Z + (8 * (int64_t)e + i) * m + j;
    *p = (zero ? 0.0 : *p) + acc[i];
  }
}

// K = P C P^T: entry (8 c + i, 8 c' + i') sums the injection coefficients of the
// two fine corners with the coarse block of their parents.
__global__ __launch_bounds__(kThreads) void k_mg3_dense_coarse(int n, const double* __restrict__ C,
                                                               double* __restrict__ K) {
  const int64_t m = 8 * (int64_t)n * n * n, mc = m / 8;
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t >= m * m) return;
  const int64_t R = t / m, Cc = t % m;
  const int nc = n / 2;
  auto parent = [&](int64_t v, int& q, int& i) {
    const int64_t e = v >> 3;
    const int x = int(e % n), y = int((e / n) % n), z = int(e / ((int64_t)n * n));
    q = (x & 1) | ((y & 1) << 1) | ((z & 1) << 2);
    i = int(v & 7);
    return ((int64_t)(z >> 1) * nc + (y >> 1)) * nc + (x >> 1);
  };
  int q, i, q2, i2;
  const int64_t E = parent(R, q, i), F = parent(Cc, q2, i2);
  double acc = 0.0;
  for (int I = 0; I < 8; ++I) {
    const double pi = inject(q, i, I);
    if (pi == 0.0) continue;
    double a = 0.0;
    for (int J = 0; J < 8; ++J) a += C[(8 * E + I) * mc + 8 * F + J] * inject(q2, i2, J);
    acc += pi * a;
  }
  K[t] = acc;
}

__global__ __launch_bounds__(kThreads) void k_mg3_start(int64_t len, double* __restrict__ z,
                                                        Mg3Scalars* sc, double rel2, int max_iters) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < len;
       i += (int64_t)gridDim.x * kThreads)
    z[i] = 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc->rel2 = rel2;
    sc->thresh2 = 0.0;
    sc->rr = 0.0;
    sc->active = 1;
    sc->first = 1;
    sc->iters = 0;
    sc->max_iters = max_iters;
  }
}

__global__ __launch_bounds__(kThreads) void k_mg3_test(int nparts, const double* __restrict__ part,
                                                       Mg3Scalars* sc) {
  if (sc->active == 0) return;
  __shared__ double sh[kThreads];
  double v = 0.0;
  for (int i = threadIdx.x; i < nparts; i += kThreads) v += part[i];
  const double rr = block_sum(v, sh);
  if (threadIdx.x == 0) {
    if (sc->first) {
      sc->thresh2 = sc->rel2 * rr;
      sc->first = 0;
    }
    sc->rr = rr;
    if (!(rr > sc->thresh2) || sc->iters >= sc->max_iters)
      sc->active = 0;
    else
      sc->iters += 1;
  }
}

__global__ __launch_bounds__(kThreads) void k_mg3_scale(int64_t len, double a,
                                                        const double* __restrict__ x,
                                                        double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < len) y[i] = a * x[i];
}

unsigned cube_blocks(int64_t cubes) { return unsigned((cubes + kCubesPerBlock - 1) / kCubesPerBlock); }

// One wavefront per workgroup: the level of 16 cubes per side has 516 tasks, two
// per compute unit, where workgroups of four left half of the units idle.
unsigned task_blocks(const Mg3LevelDev& L) { return unsigned(L.tasks); }

}  // namespace

bool mg3_split(int nk) { return nk <= kSplitMaxN; }

int mg3_res_blocks(const Mg3LevelDev& L) {
  return mg3_split(L.n) ? int((8 * (int64_t)L.n * L.n * L.n + kThreads / 8 - 1) / (kThreads / 8))
                        : int(task_blocks(L));
}

hipError_t launch_mg3_res(const Mg3LevelDev& L, const double* f, const double* z, double* r,
                          double* part, const int32_t* guard, hipStream_t st) {
  if (mg3_split(L.n)) {
    hipLaunchKernelGGL(k_mg3_res_split, dim3(mg3_res_blocks(L)), dim3(kThreads), 0, st, L.n, L.op, f, z,
                       r, part, guard);
  } else {
    if (!L.cubes || L.tasks <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mg3_res, dim3(task_blocks(L)), dim3(64), 0, st, L.n, L.tasks, L.cubes,
                       L.cls, L.op, f, z, r, part, guard);
  }
  return hipGetLastError();
}

hipError_t launch_mg3_ras(const Mg3LevelDev& L, const double* r, double* z, bool zero,
                          const int32_t* guard, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (mg3_split(L.n)) {
    const int64_t outs = 8 * (int64_t)L.n * L.n * L.n;
    hipExtLaunchKernelGGL(k_mg3_ras_split, dim3(unsigned((outs + kThreads / 32 - 1) / (kThreads / 32))),
                          dim3(kThreads), 0, st, ev0, ev1, 0, L.n, L.ras, r, z, int(zero), guard);
  } else {
    if (!L.cubes || L.tasks <= 0) return hipErrorInvalidValue;
    hipExtLaunchKernelGGL(k_mg3_ras, dim3(task_blocks(L)), dim3(64), 0, st, ev0, ev1, 0, L.n,
                          L.tasks, L.cubes, L.cls, L.ras, r, z, int(zero), guard);
  }
  return hipGetLastError();
}

hipError_t launch_mg3_restrict(int nf, const double* r, double* fc, const int32_t* guard,
                               hipStream_t st) {
  const int nc = nf / 2;
  hipLaunchKernelGGL(k_mg3_restrict, dim3(cube_blocks((int64_t)nc * nc * nc)), dim3(kThreads), 0, st,
                     nf, r, fc, guard);
  return hipGetLastError();
}

hipError_t launch_mg3_prolong(int nf, const double* zc, double* z, bool assign,
                              const int32_t* guard, hipStream_t st) {
  hipLaunchKernelGGL(k_mg3_prolong, dim3(cube_blocks((int64_t)nf * nf * nf)), dim3(kThreads), 0, st,
                     nf, zc, z, int(assign), guard);
  return hipGetLastError();
}

hipError_t launch_mg3_dense(int m, const double* inv, const double* f, double* z,
                            const int32_t* guard, hipStream_t st) {
  hipLaunchKernelGGL(k_mg3_dense, dim3((m + kThreads / 64 - 1) / (kThreads / 64)), dim3(kThreads), 0, st,
                     m, inv, f, z, guard);
  return hipGetLastError();
}

hipError_t launch_mg3_res_cols(const Mg3LevelDev& L, const double* Z, double* R, hipStream_t st) {
  const int64_t m = 8 * (int64_t)L.n * L.n * L.n;
  if (!mg3_split(L.n) || m % 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mg3_res_cols, dim3(unsigned(m / 64), L.n * L.n * L.n), dim3(64), 0, st, L.n, L.op, Z, R);
  return hipGetLastError();
}

hipError_t launch_mg3_ras_cols(const Mg3LevelDev& L, const double* R, double* Z, bool zero, hipStream_t st) {
  const int64_t m = 8 * (int64_t)L.n * L.n * L.n;
  if (!mg3_split(L.n) || m % 64 || !L.ras) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mg3_ras_cols, dim3(unsigned(m / 64), L.n * L.n * L.n), dim3(64), 0, st, L.n, L.ras, R, Z,
                     int(zero));
  return hipGetLastError();
}

hipError_t launch_mg3_dense_coarse(int nk, const double* C, double* K, hipStream_t st) {
  const int64_t m = 8 * (int64_t)nk * nk * nk;
  hipLaunchKernelGGL(k_mg3_dense_coarse, dim3(unsigned((m * m + kThreads - 1) / kThreads)), dim3(kThreads),
                     0, st, nk, C, K);
  return hipGetLastError();
}

hipError_t launch_mg3_start(int64_t len, double* z, Mg3Scalars* sc, double rel2, int max_iters,
                            hipStream_t st) {
  const int64_t want = (len + kThreads - 1) / kThreads;
  const unsigned blocks = unsigned(want < 1 ? 1 : (want > 1024 ? 1024 : want));
  hipLaunchKernelGGL(k_mg3_start, dim3(blocks), dim3(kThreads), 0, st, len, z, sc, rel2, max_iters);
  return hipGetLastError();
}

hipError_t launch_mg3_test(int nparts, const double* part, Mg3Scalars* sc, hipStream_t st) {
  hipLaunchKernelGGL(k_mg3_test, dim3(1), dim3(kThreads), 0, st, nparts, part, sc);
  return hipGetLastError();
}

hipError_t launch_mg3_scale(int64_t len, double a, const double* x, double* y, hipStream_t st) {
  hipLaunchKernelGGL(k_mg3_scale, dim3(unsigned((len + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     st, len, a, x, y);
  return hipGetLastError();
}

}  // namespace dcg3

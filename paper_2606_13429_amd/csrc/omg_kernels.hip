// Kernels of the outer multigrid preconditioner (W-cycle on A*, layouts in
// omg.hpp).  Level vectors hold 16 FP64 values per square.
//
// The RAS step and the residual split every output (square, row) over a few
// lanes on levels of at most kOmgSplitMaxN squares per side (one lane per
// diamond square resp. face slot, one round of 128-byte loads each, a fixed
// shuffle sum).  Larger levels run them as FP64 MFMA products of a class table
// with the inputs of 16 squares: gathered by each wavefront for the squares of one
// class up to kOmgTaskMaxN, staged in LDS by 8 x 8 bricks above.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "host_setup.hpp"
#include "mg_common.hpp"
#include "omg.hpp"

namespace dcg {

namespace {

using mg::ld2_any;   // the caller's vectors

constexpr int D = kOmgDofs;
constexpr int kThreads = 256;

__device__ __forceinline__ int op_axis(int x, int n) { return x == 0 ? 0 : (x == n - 1 ? 2 : 1); }
__device__ __forceinline__ int ras_axis(int x, int n) {
  return x < 3 ? x : (n - 1 - x < 3 ? 6 - (n - 1 - x) : 3);
}
__device__ __forceinline__ int ras_class(int x, int y, int n) {
  return n < kOmgRasClassMinN ? y * n + x : ras_axis(x, n) + 7 * ras_axis(y, n);
}

// The 2D diamond (|dx| + |dy| <= 2), by dy then dx (omg_diamond).
struct Diamond2 {
  int d[kOmgDiamond][2];
  constexpr Diamond2() : d() {
    int k = 0;
    for (int dy = -2; dy <= 2; ++dy)
      for (int dx = -2; dx <= 2; ++dx)
        if ((dx < 0 ? -dx : dx) + (dy < 0 ? -dy : dy) <= 2) {
          d[k][0] = dx;
          d[k][1] = dy;
          ++k;
        }
  }
};

constexpr int kSlotOff[kSlots][2] = {{0, 0}, {-1, 0}, {1, 0}, {0, -1}, {0, 1}};

// ---- small levels
// RAS: 16 lanes per output (lane d < 13 takes diamond square d), 16 outputs
// per workgroup.
__global__ __launch_bounds__(kThreads) void k_omg_ras_split(int n, const double* __restrict__ ras,
                                                            const double* __restrict__ r,
                                                            double* __restrict__ z, int zero) {
  constexpr Diamond2 DM;
  const int64_t ne = (int64_t)n * n;
  const int64_t out = (int64_t)blockIdx.x * (kThreads / 16) + (threadIdx.x >> 4);
  const int d = threadIdx.x & 15;
  const int64_t e = out / D;
  const int row = int(out % D);
  double acc = 0.0;
  if (e < ne && d < kOmgDiamond) {
    const int x = int(e % n), y = int(e / n);
    const int qx = x + DM.d[d][0], qy = y + DM.d[d][1];
    if (qx >= 0 && qy >= 0 && qx < n && qy < n) {
      const double* K = ras + ((int64_t)ras_class(x, y, n) * D + row) * kOmgRasCols + D * d;
      const double* rn = r + D * ((int64_t)qy * n + qx);
#pragma unroll
      for (int b = 0; b < D; ++b) acc += K[b] * rn[b];
    }
  }
#pragma unroll
  for (int m = 8; m > 0; m >>= 1) acc += __shfl_xor(acc, m, 16);
  if (d == 0 && e < ne) z[D * e + row] = (zero ? 0.0 : z[D * e + row]) + acc;
}

// Residual: 8 lanes per output (lane s < 5 takes face slot s), 32 outputs per
// workgroup.
__global__ __launch_bounds__(kThreads) void k_omg_res_split(int n, const double* __restrict__ op,
                                                            const double* __restrict__ f,
                                                            const double* __restrict__ z,
                                                            double* __restrict__ r) {
  const int64_t ne = (int64_t)n * n;
  const int64_t out = (int64_t)blockIdx.x * (kThreads / 8) + (threadIdx.x >> 3);
  const int s = threadIdx.x & 7;
  const int64_t e = out / D;
  const int row = int(out % D);
  double acc = 0.0;
  if (e < ne && s < kSlots) {
    const int x = int(e % n), y = int(e / n);
    const int qx = x + kSlotOff[s][0], qy = y + kSlotOff[s][1];
    if (qx >= 0 && qy >= 0 && qx < n && qy < n) {
      const int cls = op_axis(x, n) + 3 * op_axis(y, n);
      const double* A = op + ((cls * kSlots + s) * D + row) * D;
      const double* zn = z + D * ((int64_t)qy * n + qx);
#pragma unroll
      for (int b = 0; b < D; ++b) acc -= A[b] * zn[b];
    }
  }
#pragma unroll
  for (int m = 4; m > 0; m >>= 1) acc += __shfl_xor(acc, m, 8);
  if (s == 0 && e < ne) r[D * e + row] = (f ? f[D * e + row] : 0.0) + acc;
}

typedef double v4d __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4d mfma64(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---- middle levels (kOmgSplitMaxN < n_k <= kOmgTaskMaxN): one wavefront per task
// of 16 squares of one class, the class's 16 rows times the squares' gathered
// inputs with v_mfma_f64_16x16x4f64, four table columns a step.  Lane l supplies
// row l % 16, column 4 s + l / 16 of the table (the operand-order tables make a
// step's operand one contiguous 512-byte run) and input value 4 s + l / 16 of
// square l % 16's window, and receives rows 4 v + l / 16 (v = 0..3) of that square.
// All operands come from L1 / L2: no LDS, no barrier, and boundary tasks cost what
// interior ones do.  A RAS step takes 5.5 / 6.5 / 12.3 us and a residual 3.5 / 4.1 /
// 6.6 us at n = 32 / 64 / 128, where the split kernels (32) took 8.7 and 4.8 us and
// the bricks below 19.7 / 20.7 and 8.8 / 8.7 us; at 256 the gathers, 16 lanes in 16
// cache lines, make it 37 us against the bricks' 27.5 us.
struct Task {
  int q, cls, x, y, e;   // lane group, RAS class, the lane's square
  bool valid;
};

// Workgroups go round robin to the 8 XCDs: each takes a contiguous run of tasks.
__device__ __forceinline__ Task load_task(int n, const int32_t* __restrict__ squares,
                                          const int32_t* __restrict__ cls, int tasks) {
  const int b = blockIdx.x, per = tasks >> 3;
  const int id = b < 8 * per ? (b & 7) * per + (b >> 3) : b;
  Task t;
  t.q = threadIdx.x >> 4;
  t.cls = cls[id];
  const int e = squares[16 * id + (threadIdx.x & 15)];
  t.valid = e >= 0;
  t.e = e >= 0 ? e : ~e;   // padding repeats a square of the task
  t.x = t.e % n;
  t.y = t.e / n;
  return t;
}

// The four table steps of each of the NB neighbours at OFF; loads are
// unconditional (from the square itself outside the domain).
template <int NB, typename OFF>
__device__ __forceinline__ v4d task_products(const Task& t, int n, OFF off, const double* __restrict__ A,
                                             const double* __restrict__ v) {
  double u[NB][4];
#pragma unroll
  for (int d = 0; d < NB; ++d) {
    const int dx = off(d, 0), dy = off(d, 1);
    const bool in = t.x + dx >= 0 && t.y + dy >= 0 && t.x + dx < n && t.y + dy < n;
    const double* p = v + D * (int64_t)(t.e + (in ? dy * n + dx : 0)) + t.q;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double x = p[4 * s];
      u[d][s] = in ? x : 0.0;
    }
  }
  v4d a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0;
#pragma unroll
  for (int d = 0; d < NB; ++d) {
    a0 = mfma64(A[64 * (4 * d)], u[d][0], a0);
    a1 = mfma64(A[64 * (4 * d + 1)], u[d][1], a1);
    a0 = mfma64(A[64 * (4 * d + 2)], u[d][2], a0);
    a1 = mfma64(A[64 * (4 * d + 3)], u[d][3], a1);
  }
  return a0 + a1;
}

__global__ __launch_bounds__(64) void k_omg_ras(int n, int tasks, const int32_t* __restrict__ squares,
                                                const int32_t* __restrict__ cls,
                                                const double* __restrict__ rasm,
                                                const double* __restrict__ r, double* __restrict__ z,
                                                int zero) {
  const Task t = load_task(n, squares, cls, tasks);
  constexpr Diamond2 DM;
  auto off = [&](int d, int a) { return DM.d[d][a]; };
  double zv[4];
  double* zp = z + D * (int64_t)t.e + t.q;
#pragma unroll
  for (int v = 0; v < 4; ++v) zv[v] = zero ? 0.0 : zp[4 * v];
  const double* A = rasm + (int64_t)t.cls * kOmgRasSteps * 64 + threadIdx.x;
  const v4d a = task_products<kOmgDiamond>(t, n, off, A, r);
  if (t.valid)
#pragma unroll
    for (int v = 0; v < 4; ++v) zp[4 * v] = zv[v] + a[v];
}

__global__ __launch_bounds__(64) void k_omg_res(int n, int tasks, const int32_t* __restrict__ squares,
                                                const int32_t* __restrict__ cls,
                                                const double* __restrict__ opm,
                                                const double* __restrict__ f,
                                                const double* __restrict__ z, double* __restrict__ r) {
  const Task t = load_task(n, squares, cls, tasks);
  auto off = [&](int s, int a) { return kSlotOff[s][a]; };
  // operator class: 0 low side, 2 high side, 1 inside of the distance class
  const int px = t.cls % 7, py = t.cls / 7;
  const int oc = (px == 0 ? 0 : (px == 6 ? 2 : 1)) + 3 * (py == 0 ? 0 : (py == 6 ? 2 : 1));
  double fv[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) fv[v] = f ? f[D * (int64_t)t.e + 4 * v + t.q] : 0.0;
  const double* A = opm + (int64_t)oc * kOmgOpSteps * 64 + threadIdx.x;
  const v4d a = task_products<kSlots>(t, n, off, A, z);
  if (t.valid)
#pragma unroll
    for (int v = 0; v < 4; ++v) r[D * (int64_t)t.e + 4 * v + t.q] = fv[v] - a[v];
}

// ---- large levels: 8 x 8 bricks with their input staged in LDS
constexpr int kBrick = 8;

template <int H>
struct Box2 {
  static constexpr int X = kBrick + 2 * H;
  static constexpr int N = X * X;
  static constexpr int S = N + 1;   // component stride (padding spreads the banks)
};

template <int H>
__device__ __forceinline__ void stage_box(int n, int x0, int y0, const double* __restrict__ v,
                                          double* lds) {
  using B = Box2<H>;
  for (int i = threadIdx.x; i < B::N * D; i += blockDim.x) {
    const int c = i / D, b = i % D;
    const int x = x0 - H + c % B::X, y = y0 - H + c / B::X;
    double val = 0.0;
    if (x >= 0 && y >= 0 && x < n && y < n) val = v[D * ((int64_t)y * n + x) + b];
    lds[b * B::S + c] = val;
  }
}

// ---- MFMA form: on an 8 x 8 brick the step is a class table (16 rows) times
// the gathered inputs of the brick's squares, 16 squares per wavefront as the
// columns of v_mfma_f64_16x16x4f64, four table columns a step.  Lane l
// supplies row l % 16, column 4 s + l / 16 of the table (the operand-order
// tables make one step's operand one contiguous 512-byte run) and, for square
// l % 16 of its wavefront, input value 4 s + l / 16 of that square's window
// from LDS; it receives rows 4 v + l / 16 (v = 0..3) of square l % 16.
// Interior bricks (every square of the interior class) stage the one class
// table in LDS next to the input and run the products from LDS with two
// accumulators; boundary bricks, dispatched first, take the distinct classes
// of each wavefront one after the other with the table read from global
// memory, keeping for each square the product with its own class.
constexpr int kMfmaThreads = 256;   // 4 wavefronts x 16 squares = one brick

struct MfmaLane {
  int x0, y0, x, y, q, o1, o2;   // brick, square, output row group, LDS offsets (halo 1 / 2)
  bool interior;
  int64_t e;
};

// Workgroup -> brick: the ring of boundary bricks first, then the interior.
__device__ __forceinline__ MfmaLane mfma_lane(int n) {
  const int nb = n / kBrick, ring = nb > 1 ? 4 * (nb - 1) : 1;
  const int b = blockIdx.x;
  int bx, by;
  if (b < ring) {
    if (b < nb) {
      bx = b;
      by = 0;
    } else if (b < 2 * nb) {
      bx = b - nb;
      by = nb - 1;
    } else {
      const int t = b - 2 * nb;
      bx = t < nb - 2 ? 0 : nb - 1;
      by = 1 + (t < nb - 2 ? t : t - (nb - 2));
    }
  } else {
    const int t = b - ring;
    bx = 1 + t % (nb - 2);
    by = 1 + t / (nb - 2);
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = lane & 15, lx = j & 7, ly = 2 * w + (j >> 3);
  MfmaLane L;
  L.x0 = bx * kBrick;
  L.y0 = by * kBrick;
  L.interior = b >= ring;
  L.x = L.x0 + lx;
  L.y = L.y0 + ly;
  L.q = lane >> 4;
  L.o1 = (ly + 1) * Box2<1>::X + lx + 1;
  L.o2 = (ly + 2) * Box2<2>::X + lx + 2;
  L.e = (int64_t)L.y * n + L.x;
  return L;
}

// Copies one class table (steps x 64 doubles, operand order) into LDS.
template <int STEPS>
__device__ __forceinline__ void stage_table(const double* __restrict__ src, double* kt) {
  for (int i = threadIdx.x; i < STEPS * 64; i += kMfmaThreads) kt[i] = src[i];
}

// RAS products over the 13-square diamond: Kv(s) is the lane's table operand
// of step s, the input of step s the LDS plane 4 (s % 4) + q at the square's
// offset plus the diamond offset of s / 4.
template <typename KV>
__device__ __forceinline__ v4d ras_chain(KV Kv, const double* rs, const MfmaLane& L, v4d t) {
  using B = Box2<2>;
  constexpr Diamond2 DM;
  v4d t1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int d = 0; d < kOmgDiamond; ++d) {
    const int od = DM.d[d][1] * B::X + DM.d[d][0];
    t = mfma64(Kv(4 * d), rs[(0 + L.q) * B::S + L.o2 + od], t);
    t1 = mfma64(Kv(4 * d + 1), rs[(4 + L.q) * B::S + L.o2 + od], t1);
    t = mfma64(Kv(4 * d + 2), rs[(8 + L.q) * B::S + L.o2 + od], t);
    t1 = mfma64(Kv(4 * d + 3), rs[(12 + L.q) * B::S + L.o2 + od], t1);
  }
  return t + t1;
}

template <typename KV>
__device__ __forceinline__ v4d res_chain(KV Kv, const double* zs, const MfmaLane& L) {
  using B = Box2<1>;
  v4d t = {0.0, 0.0, 0.0, 0.0}, t1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int sl = 0; sl < kSlots; ++sl) {
    const int os = kSlotOff[sl][1] * B::X + kSlotOff[sl][0];
    t = mfma64(Kv(4 * sl), zs[(0 + L.q) * B::S + L.o1 + os], t);
    t1 = mfma64(Kv(4 * sl + 1), zs[(4 + L.q) * B::S + L.o1 + os], t1);
    t = mfma64(Kv(4 * sl + 2), zs[(8 + L.q) * B::S + L.o1 + os], t);
    t1 = mfma64(Kv(4 * sl + 3), zs[(12 + L.q) * B::S + L.o1 + os], t1);
  }
  return t + t1;
}

// Boundary bricks: the lanes of a wavefront take squares of as few classes as
// possible -- square slot i of the brick (wavefront i / 16, lane i % 16) gets
// the square of rank i in the order (class, position) -- so that an edge brick
// needs at most two class trips per wavefront.  cls_of(x, y) is the class.
template <typename CF>
__device__ __forceinline__ void sort_squares(MfmaLane& L, int n, CF cls_of, int* scls, int* sperm) {
  if (threadIdx.x < kBrick * kBrick)
    scls[threadIdx.x] = cls_of(L.x0 + (threadIdx.x & 7), L.y0 + (threadIdx.x >> 3));
  __syncthreads();
  if (threadIdx.x < kBrick * kBrick) {
    const int me = threadIdx.x, c = scls[me];
    int rank = 0;
    for (int i = 0; i < kBrick * kBrick; ++i) {
      const int ci = scls[i];
      rank += (ci < c) || (ci == c && i < me);
    }
    sperm[rank] = me;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, sq = sperm[16 * (threadIdx.x >> 6) + (lane & 15)];
  const int lx = sq & 7, ly = sq >> 3;
  L.x = L.x0 + lx;
  L.y = L.y0 + ly;
  L.o1 = (ly + 1) * Box2<1>::X + lx + 1;
  L.o2 = (ly + 2) * Box2<2>::X + lx + 2;
  L.e = (int64_t)L.y * n + L.x;
}

// three workgroups fit a compute unit's LDS; registers are kept to match
__global__ __launch_bounds__(kMfmaThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_omg_ras_m(int n, const double* __restrict__ rasm,
                                                            const double* __restrict__ r,
                                                            double* __restrict__ z, int zero) {
  using B = Box2<2>;
  __shared__ double rs[D * B::S];
  __shared__ double kt[kOmgRasSteps * 64];
  __shared__ int scls[kBrick * kBrick], sperm[kBrick * kBrick];
  MfmaLane L = mfma_lane(n);
  const int lane = threadIdx.x & 63;
  if (L.interior) stage_table<kOmgRasSteps>(rasm + (int64_t)kOmgRasInterior * kOmgRasSteps * 64, kt);
  stage_box<2>(n, L.x0, L.y0, r, rs);
  if (!L.interior) sort_squares(L, n, [n](int x, int y) { return ras_class(x, y, n); }, scls, sperm);
  v4d acc;
#pragma unroll
  for (int v = 0; v < 4; ++v) acc[v] = zero ? 0.0 : z[D * L.e + 4 * v + L.q];
  __syncthreads();
  if (L.interior) {
    acc = ras_chain([&](int st) { return kt[lane + 64 * st]; }, rs, L, acc);
  } else {
    const int cls = ras_class(L.x, L.y, n);
    uint64_t pending = __ballot(true);
    while (pending) {   // the wavefront's distinct classes, one per trip
      const int c = __builtin_amdgcn_readfirstlane(__shfl(cls, __builtin_ctzll(pending), 64));
      const double* K = rasm + (int64_t)c * kOmgRasSteps * 64 + lane;
      double a[kOmgRasSteps];   // the trip's operands requested ahead of the products
#pragma unroll
      for (int st = 0; st < kOmgRasSteps; ++st) a[st] = K[64 * st];
      const v4d t = ras_chain([&](int st) { return a[st]; }, rs, L, acc);
      const bool mine = cls == c;
      if (mine) acc = t;
      pending &= ~__ballot(mine);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) z[D * L.e + 4 * v + L.q] = acc[v];
}

__global__ __launch_bounds__(kMfmaThreads) void k_omg_res_m(int n, const double* __restrict__ opm,
                                                            const double* __restrict__ f,
                                                            const double* __restrict__ z,
                                                            double* __restrict__ r) {
  using B = Box2<1>;
  __shared__ double zs[D * B::S];
  __shared__ double kt[kOmgOpSteps * 64];
  __shared__ int scls[kBrick * kBrick], sperm[kBrick * kBrick];
  MfmaLane L = mfma_lane(n);
  const int lane = threadIdx.x & 63;
  if (L.interior) stage_table<kOmgOpSteps>(opm + (int64_t)kOmgOpInterior * kOmgOpSteps * 64, kt);
  stage_box<1>(n, L.x0, L.y0, z, zs);
  if (!L.interior)
    sort_squares(L, n, [n](int x, int y) { return op_axis(x, n) + 3 * op_axis(y, n); }, scls, sperm);
  double fv[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) fv[v] = f ? f[D * L.e + 4 * v + L.q] : 0.0;
  __syncthreads();
  v4d acc;
  if (L.interior) {
    acc = res_chain([&](int st) { return kt[lane + 64 * st]; }, zs, L);
  } else {
    const int cls = op_axis(L.x, n) + 3 * op_axis(L.y, n);
    acc = v4d{0.0, 0.0, 0.0, 0.0};
    uint64_t pending = __ballot(true);
    while (pending) {
      const int c = __builtin_amdgcn_readfirstlane(__shfl(cls, __builtin_ctzll(pending), 64));
      const double* K = opm + (int64_t)c * kOmgOpSteps * 64 + lane;
      double a[kOmgOpSteps];
#pragma unroll
      for (int st = 0; st < kOmgOpSteps; ++st) a[st] = K[64 * st];
      const v4d t = res_chain([&](int st) { return a[st]; }, zs, L);
      const bool mine = cls == c;
      if (mine) acc = t;
      pending &= ~__ballot(mine);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) r[D * L.e + 4 * v + L.q] = fv[v] - acc[v];
}

// ---- transfers: one thread per (square, dof); every component injected alike
__device__ __forceinline__ double inject(int q, int i, int J) {
  double v = 1.0;
#pragma unroll
  for (int ax = 0; ax < 2; ++ax) {
    const double t = 0.5 * (((q >> ax) & 1) + ((i >> ax) & 1));
    v *= ((J >> ax) & 1) ? t : 1.0 - t;
  }
  return v;
}

__global__ __launch_bounds__(kThreads) void k_omg_restrict(int nf, const double* __restrict__ r,
                                                           double* __restrict__ fc) {
  const int nc = nf / 2;
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t >= (int64_t)D * nc * nc) return;
  const int64_t E = t / D;
  const int dof = int(t % D), c = dof >> 2, J = dof & 3;
  const int X = int(E % nc), Y = int(E / nc);
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double* rc = r + D * ((int64_t)(2 * Y + (q >> 1)) * nf + 2 * X + (q & 1)) + 4 * c;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc += inject(q, i, J) * rc[i];
  }
  fc[t] = acc;
}

__global__ __launch_bounds__(kThreads) void k_omg_prolong(int nf, const double* __restrict__ zc,
                                                          double* __restrict__ z, int assign) {
  const int nc = nf / 2;
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t >= (int64_t)D * nf * nf) return;
  const int64_t e = t / D;
  const int dof = int(t % D), c = dof >> 2, i = dof & 3;
  const int x = int(e % nf), y = int(e / nf);
  const int q = (x & 1) | ((y & 1) << 1);
  const double* zE = zc + D * ((int64_t)(y >> 1) * nc + (x >> 1)) + 4 * c;
  double acc = 0.0;
#pragma unroll
  for (int J = 0; J < 4; ++J) acc += inject(q, i, J) * zE[J];
  z[t] = assign ? acc : z[t] + acc;
}

// z = A f, A dense m x m (m even): one wavefront per row, lanes over pairs of
// columns, a fixed shuffle sum.  Bound by the matrix (134 MB at m = 4096).
__global__ __launch_bounds__(kThreads) void k_omg_dense(int m, const double* __restrict__ A,
                                                        const double* __restrict__ f,
                                                        double* __restrict__ z) {
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
// once (set-up): thread (square, column), the table rows through scalar loads, the
// columns of a wavefront contiguous.  R = I - A* Z (Z = NULL: R = I).
__global__ __launch_bounds__(kThreads) void k_omg_res_cols(int n, const double* __restrict__ op,
                                                           const double* __restrict__ Z,
                                                           double* __restrict__ R) {
  const int64_t m = D * (int64_t)n * n;
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int e = blockIdx.y, x = e % n, y = e / n;
  const int cls = op_axis(x, n) + 3 * op_axis(y, n);
  double acc[D];
#pragma unroll
  for (int i = 0; i < D; ++i) acc[i] = D * (int64_t)e + i == j ? 1.0 : 0.0;
  for (int s = 0; Z && s < kSlots; ++s) {
    const int qx = x + kSlotOff[s][0], qy = y + kSlotOff[s][1];
    if (qx < 0 || qy < 0 || qx >= n || qy >= n) continue;
    const double* B = op + (cls * kSlots + s) * D * D;
#pragma unroll 4
    for (int b = 0; b < D; ++b) {
      const double v = Z[(D * ((int64_t)qy * n + qx) + b) * m + j];
#pragma unroll
      for (int i = 0; i < D; ++i) acc[i] -= B[D * i + b] * v;
    }
  }
#pragma unroll
  for (int i = 0; i < D; ++i) R[(D * (int64_t)e + i) * m + j] = acc[i];
}

// Z = (zero ? 0 : Z) + S R.
__global__ __launch_bounds__(kThreads) void k_omg_ras_cols(int n, const double* __restrict__ ras,
                                                           const double* __restrict__ R,
                                                           double* __restrict__ Z, int zero) {
  constexpr Diamond2 DM;
  const int64_t m = D * (int64_t)n * n;
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int e = blockIdx.y, x = e % n, y = e / n;
  const double* K = ras + (int64_t)ras_class(x, y, n) * D * kOmgRasCols;
  double acc[D];
#pragma unroll
  for (int i = 0; i < D; ++i) acc[i] = 0.0;
  for (int d = 0; d < kOmgDiamond; ++d) {
    const int qx = x + DM.d[d][0], qy = y + DM.d[d][1];
    if (qx < 0 || qy < 0 || qx >= n || qy >= n) continue;
#pragma unroll 4
    for (int b = 0; b < D; ++b) {
      const double v = R[(D * ((int64_t)qy * n + qx) + b) * m + j];
#pragma unroll
      for (int i = 0; i < D; ++i) acc[i] += K[kOmgRasCols * i + D * d + b] * v;
    }
  }
#pragma unroll
  for (int i = 0; i < D; ++i) {
    double* z = Z + (D * (int64_t)e + i) * m + j;
    *z = (zero ? 0.0 : *z) + acc[i];
  }
}

// K = P C P^T: entry (16 e + 4 c + i, 16 e' + 4 c' + i') sums the injection
// coefficients of the two fine corners with the coarse block of their parents.
__global__ __launch_bounds__(kThreads) void k_omg_dense_coarse(int n, const double* __restrict__ C,
                                                               double* __restrict__ K) {
  const int64_t m = D * (int64_t)n * n, mc = m / 4;
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t >= m * m) return;
  const int nc = n / 2;
  auto parent = [&](int64_t v, int& q, int& i) {   // first coarse dof of the component
    const int64_t e = v / D;
    const int x = int(e % n), y = int(e / n), dof = int(v % D);
    q = (x & 1) | ((y & 1) << 1);
    i = dof & 3;
    return D * ((int64_t)(y >> 1) * nc + (x >> 1)) + 4 * (dof >> 2);
  };
  int q, i, q2, i2;
  const int64_t E = parent(t / m, q, i), F = parent(t % m, q2, i2);
  double acc = 0.0;
  for (int I = 0; I < 4; ++I) {
    double a = 0.0;
    for (int J = 0; J < 4; ++J) a += C[(E + I) * mc + F + J] * inject(q2, i2, J);
    acc += inject(q, i, I) * a;
  }
  K[t] = acc;
}

unsigned bricks(int nk) { return unsigned((nk / kBrick) * (nk / kBrick)); }
unsigned blocks_for(int64_t threads) { return unsigned((threads + kThreads - 1) / kThreads); }

}  // namespace

hipError_t launch_omg_res(const OmgLevelDev& L, const double* f, const double* z, double* r,
                          hipStream_t st) {
  if (L.n <= kOmgSplitMaxN) {
    hipLaunchKernelGGL(k_omg_res_split, dim3(blocks_for(8 * (int64_t)D * L.n * L.n)), dim3(kThreads), 0, st,
                       L.n, L.op, f, z, r);
  } else if (L.n <= kOmgTaskMaxN) {
    if (!L.squares || L.tasks <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_omg_res, dim3(L.tasks), dim3(64), 0, st, L.n, L.tasks, L.squares, L.cls, L.opm, f,
                       z, r);
  } else {
    if (L.n % kBrick) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_omg_res_m, dim3(bricks(L.n)), dim3(kMfmaThreads), 0, st, L.n, L.opm, f, z, r);
  }
  return hipGetLastError();
}

hipError_t launch_omg_ras(const OmgLevelDev& L, const double* r, double* z, bool zero, hipStream_t st,
                          hipEvent_t ev0, hipEvent_t ev1) {
  if (L.n <= kOmgSplitMaxN) {
    hipExtLaunchKernelGGL(k_omg_ras_split, dim3(blocks_for(16 * (int64_t)D * L.n * L.n)), dim3(kThreads), 0,
                          st, ev0, ev1, 0, L.n, L.ras, r, z, int(zero));
  } else if (L.n <= kOmgTaskMaxN) {
    if (!L.squares || L.tasks <= 0) return hipErrorInvalidValue;
    hipExtLaunchKernelGGL(k_omg_ras, dim3(L.tasks), dim3(64), 0, st, ev0, ev1, 0, L.n, L.tasks, L.squares,
                          L.cls, L.rasm, r, z, int(zero));
  } else {
    if (L.n % kBrick) return hipErrorInvalidValue;
    hipExtLaunchKernelGGL(k_omg_ras_m, dim3(bricks(L.n)), dim3(kMfmaThreads), 0, st, ev0, ev1, 0, L.n,
                          L.rasm, r, z, int(zero));
  }
  return hipGetLastError();
}

hipError_t launch_omg_res_cols(const OmgLevelDev& L, const double* Z, double* R, hipStream_t st) {
  const int64_t m = D * (int64_t)L.n * L.n;
  if (L.n > kOmgSplitMaxN || m % kThreads) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_omg_res_cols, dim3(unsigned(m / kThreads), L.n * L.n), dim3(kThreads), 0, st, L.n,
                     L.op, Z, R);
  return hipGetLastError();
}

hipError_t launch_omg_ras_cols(const OmgLevelDev& L, const double* R, double* Z, bool zero, hipStream_t st) {
  const int64_t m = D * (int64_t)L.n * L.n;
  if (L.n > kOmgSplitMaxN || m % kThreads || !L.ras) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_omg_ras_cols, dim3(unsigned(m / kThreads), L.n * L.n), dim3(kThreads), 0, st, L.n,
                     L.ras, R, Z, int(zero));
  return hipGetLastError();
}

hipError_t launch_omg_dense_coarse(int nk, const double* C, double* K, hipStream_t st) {
  const int64_t m = D * (int64_t)nk * nk;
  hipLaunchKernelGGL(k_omg_dense_coarse, dim3(blocks_for(m * m)), dim3(kThreads), 0, st, nk, C, K);
  return hipGetLastError();
}

hipError_t launch_omg_restrict(int nf, const double* r, double* fc, hipStream_t st) {
  const int nc = nf / 2;
  hipLaunchKernelGGL(k_omg_restrict, dim3(blocks_for((int64_t)D * nc * nc)), dim3(kThreads), 0, st, nf, r,
                     fc);
  return hipGetLastError();
}

hipError_t launch_omg_prolong(int nf, const double* zc, double* z, bool assign, hipStream_t st) {
  hipLaunchKernelGGL(k_omg_prolong, dim3(blocks_for((int64_t)D * nf * nf)), dim3(kThreads), 0, st, nf, zc,
                     z, int(assign));
  return hipGetLastError();
}

hipError_t launch_omg_dense(int m, const double* inv, const double* f, double* z, hipStream_t st) {
  hipLaunchKernelGGL(k_omg_dense, dim3(unsigned((m + kThreads / 64 - 1) / (kThreads / 64))), dim3(kThreads),
                     0, st, m, inv, f, z);
  return hipGetLastError();
}

}  // namespace dcg

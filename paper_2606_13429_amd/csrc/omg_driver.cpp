// The outer multigrid preconditioner of a solver handle (omg.hpp): set-up of
// the A* hierarchy on the device, B(r) = Wcycle_J(r, 0) (Algorithm 4 on the
// hierarchy of A*, replayed as one captured HIP graph), and its level
// operators for dcg_apply.
#include <hip/hip_runtime.h>

#include <cstring>
#include <vector>

#include "kernels.hpp"
#include "omg.hpp"
#include "runtime.hpp"

namespace dcg {

namespace {

constexpr int D = kOmgDofs;

template <typename T>
T* upload(Workspace& ws, const std::vector<T>& v) {
  T* d = static_cast<T*>(ws.alloc(v.size() * sizeof(T)));
  DCG_HIP(hipMemcpy(d, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return d;
}

enum { kZero = 0, kWarm = 1 };

int64_t level_len(const OuterMg& g, int k) { return (int64_t)D * g.n[k - 1] * g.n[k - 1]; }

void copy(const double* x, double* y, int64_t len, hipStream_t st) {
  if (x != y) DCG_HIP(hipMemcpyAsync(y, x, len * sizeof(double), hipMemcpyDeviceToDevice, st));
}

// The W-cycle on level k for f_k = g.f[k-1] into z_k = g.z[k-1].
void cycle(const OuterMg& g, int k, int mode, hipStream_t st) {
  const int i = k - 1, nk = g.n[i];
  if (k == 1) {
    DCG_HIP(launch_omg_dense(int(level_len(g, 1)), g.cinv, g.f[0], g.z[0], st));
    return;
  }
  for (int s = 0; s < g.m; ++s) {
    if (s == 0 && mode == kZero) {
      DCG_HIP(launch_omg_ras(g.lev[i], g.f[i], g.z[i], true, st));
      continue;
    }
    DCG_HIP(launch_omg_res(g.lev[i], g.f[i], g.z[i], g.r[i], st));
    DCG_HIP(launch_omg_ras(g.lev[i], g.r[i], g.z[i], false, st));
  }
  DCG_HIP(launch_omg_res(g.lev[i], g.f[i], g.z[i], g.r[i], st));
  DCG_HIP(launch_omg_restrict(nk, g.r[i], g.f[i - 1], st));
  if (g.fold[i - 1]) {                        // both coarse cycles as one matrix
    DCG_HIP(launch_omg_dense(int(level_len(g, k - 1)), g.fold[i - 1], g.f[i - 1], g.z[i - 1], st));
  } else {
    cycle(g, k - 1, kZero, st);                 // gamma = 2 coarse cycles,
    if (k - 1 > 1) cycle(g, k - 1, kWarm, st);  // the exact solve once
  }
  DCG_HIP(launch_omg_prolong(nk, g.z[i - 1], g.z[i], false, st));
  for (int s = 0; s < g.m; ++s) {
    DCG_HIP(launch_omg_res(g.lev[i], g.f[i], g.z[i], g.r[i], st));
    DCG_HIP(launch_omg_ras(g.lev[i], g.r[i], g.z[i], false, st));
  }
}

// FoldCheck of the matrix C of level k.  At n = 32 the distance is 0.5 to 1.3 times the
// steps' rounding for dt <= 1e-2, 2 to 50 times at dt = 1 (m = 6 .. 1) and some
// thousand times at dt = 100.
bool matrix_holds(const OuterMg& g, int k, const double* C) {
  const int i = k - 1, m = int(level_len(g, k)), mp = int(level_len(g, k + 1));
  const hipStream_t st = nullptr;
  std::vector<double> a(m), a3(m), c(m);
  auto steps = [&](std::vector<double>& out) {
    cycle(g, k, kZero, st);
    cycle(g, k, kWarm, st);
    DCG_HIP(hipMemcpy(out.data(), g.z[i], m * sizeof(double), hipMemcpyDeviceToHost));
  };
  FoldCheck check;
  for (unsigned probe = 0; probe < 8; ++probe) {
    const std::vector<double> f = fold_probe(mp, probe);
    DCG_HIP(hipMemcpy(g.f[i + 1], f.data(), mp * sizeof(double), hipMemcpyHostToDevice));
    for (int s = 0; s < g.m; ++s) {
      if (s > 0) DCG_HIP(launch_omg_res(g.lev[i + 1], g.f[i + 1], g.z[i + 1], g.r[i + 1], st));
      DCG_HIP(launch_omg_ras(g.lev[i + 1], s > 0 ? g.r[i + 1] : g.f[i + 1], g.z[i + 1], s == 0, st));
    }
    DCG_HIP(launch_omg_res(g.lev[i + 1], g.f[i + 1], g.z[i + 1], g.r[i + 1], st));
    DCG_HIP(launch_omg_restrict(g.n[i + 1], g.r[i + 1], g.f[i], st));
    DCG_HIP(launch_omg_dense(m, C, g.f[i], g.r[i], st));
    DCG_HIP(hipMemcpy(c.data(), g.r[i], m * sizeof(double), hipMemcpyDeviceToHost));
    steps(a);
    DCG_HIP(launch_scale(m, 3.0, g.f[i], g.r[i], st));
    copy(g.r[i], g.f[i], m, st);
    steps(a3);
    check.add(m, [](int j) { return j; }, a, a3, c);
  }
  return check.holds();
}

// The two coarse cycles that level k gives its parent (Algorithm 4: from zero,
// then from the first's result) as one matrix, on levels of at most
// kOmgFoldMaxDofs unknowns: the cycles of the columns of the identity, step by step
// (2 W - W A* W with one cycle W in powers of I - S A* was up to 10 times further
// from the exact map at dt = 1).  The level of 16 x 16 squares is 134 MB, read in
// about 21 us, against 2 (4 m + 3) + 2 launches of 3-4 us; the next one would be
// 2.1 GB, slower than its steps.  The cycle runs the steps of a level that has no
// matrix: where the memory of the matrix or of its scratch (403 MB during set-up)
// cannot be had, or where the matrix is less accurate than they are (matrix_holds).
void fold_level(OuterMg& g, int k, Workspace& ws) {
  const int i = k - 1;
  const int64_t m = level_len(g, k);
  if (m > kOmgFoldMaxDofs || g.n[i] > kOmgSplitMaxN || (k > 2 && !g.fold[i - 1])) return;
  struct Temp {
    double* p = nullptr;
    ~Temp() { (void)hipFree(p); }
  } tmp;
  tmp.p = static_cast<double*>(try_device_alloc(3 * m * m * sizeof(double)));
  double* Z = tmp.p ? static_cast<double*>(ws.try_alloc(m * m * sizeof(double))) : nullptr;
  if (!Z) return;
  double *R = tmp.p, *K = R + m * m, *T = K + m * m;
  const hipStream_t st = nullptr;
  DCG_HIP(launch_omg_dense_coarse(g.n[i], k == 2 ? g.cinv : g.fold[i - 1], K, st));
  bool zero = true;
  auto smooth = [&]() {
    for (int s = 0; s < g.m; ++s, zero = false) {
      DCG_HIP(launch_omg_res_cols(g.lev[i], zero ? nullptr : Z, R, st));
      DCG_HIP(launch_omg_ras_cols(g.lev[i], R, Z, zero, st));
    }
  };
  for (int c = 0; c < 2; ++c) {        // two swaps: Z ends where it began
    smooth();
    DCG_HIP(launch_omg_res_cols(g.lev[i], Z, R, st));
    DCG_HIP(launch_gemm(int(m), K, R, T, Z, st));   // Z + P C P^T R
    std::swap(Z, T);
    smooth();
  }
  DCG_HIP(hipStreamSynchronize(st));
  if (matrix_holds(g, k, Z))
    g.fold[i] = Z;
  else
    ws.free_last(Z, m * m * sizeof(double));
}

}  // namespace

OuterMg::~OuterMg() {
  if (graph) (void)hipGraphExecDestroy(graph);
}

void omg_setup(dcg_ctx* h) {
  Workspace& ws = h->ws;
  const OmgHierarchy H = build_omg(h->mesh->n, h->mp.penalty, h->dt, h->nu);
  auto g = std::make_unique<OuterMg>();
  g->J = int(H.lev.size());
  g->m = h->opt.outer_mg;
  for (int k = 1; k <= g->J; ++k) {
    const OmgLevel& L = H.lev[k - 1];
    const int64_t len = (int64_t)D * L.n * L.n;
    g->n.push_back(L.n);
    g->op.push_back(upload(ws, L.op));
    g->ras.push_back(k >= 2 ? upload(ws, L.ras) : nullptr);
    g->opm.push_back(upload(ws, omg_operand_order(omg_op_rows(L.op), kOmgOpClasses, kOmgOpCols)));
    g->rasm.push_back(k >= 2 ? upload(ws, omg_operand_order(L.ras, kOmgRasClasses, kOmgRasCols)) : nullptr);
    g->f.push_back(static_cast<double*>(ws.alloc(len * sizeof(double))));
    g->z.push_back(static_cast<double*>(ws.alloc(len * sizeof(double))));
    g->r.push_back(static_cast<double*>(ws.alloc(len * sizeof(double))));
    OmgLevelDev d;
    d.n = L.n;
    d.op = g->op.back();
    d.ras = g->ras.back();
    d.opm = g->opm.back();
    d.rasm = g->rasm.back();
    if (L.n > kOmgSplitMaxN && L.n <= kOmgTaskMaxN) {
      std::vector<int32_t> squares, cls;
      omg_tasks(L.n, squares, cls);
      d.squares = upload(ws, squares);
      d.cls = upload(ws, cls);
      d.tasks = int(cls.size());
    }
    g->lev.push_back(d);
  }
  g->cinv = upload(ws, H.coarse_inv);
  g->zp = static_cast<double*>(ws.alloc((int64_t)D * g->n[g->J - 1] * g->n[g->J - 1] * sizeof(double)));
  g->fold.assign(g->J, nullptr);
  for (int k = 2; k < g->J; ++k) fold_level(*g, k, ws);
  h->omg = std::move(g);
}

// z = B r on the finest level; replayed from a graph captured on first use.
void omg_apply(dcg_ctx* h, const double* r, double* z, hipStream_t st) {
  OuterMg& g = *h->omg;
  const int J = g.J;
  const int64_t len = level_len(g, J);
  if (!h->opt.use_graph) {
    copy(r, g.f[J - 1], len, st);
    cycle(g, J, kZero, st);
    copy(g.z[J - 1], z, len, st);
    return;
  }
  if (!g.graph || g.g_in != r || g.g_out != z) {
    if (g.graph) {
      DCG_HIP(hipGraphExecDestroy(g.graph));
      g.graph = nullptr;
    }
    hipGraph_t gr = nullptr;
    DCG_HIP(hipStreamBeginCapture(h->capture_stream, hipStreamCaptureModeThreadLocal));
    try {
      copy(r, g.f[J - 1], len, h->capture_stream);
      cycle(g, J, kZero, h->capture_stream);
      copy(g.z[J - 1], z, len, h->capture_stream);
    } catch (...) {
      (void)hipStreamEndCapture(h->capture_stream, &gr);
      if (gr) (void)hipGraphDestroy(gr);
      throw;
    }
    DCG_HIP(hipStreamEndCapture(h->capture_stream, &gr));
    const hipError_t e = hipGraphInstantiate(&g.graph, gr, nullptr, nullptr, 0);
    (void)hipGraphDestroy(gr);
    DCG_HIP(e);
    g.g_in = r;
    g.g_out = z;
  }
  DCG_HIP(hipGraphLaunch(g.graph, st));
}

void omg_apply_level(dcg_ctx* h, dcg_op op, int k, const double* in, const double* in2, double* out,
                     hipStream_t st) {
  if (!h->omg) throw Error(DCG_EINVAL, "the handle has no outer multigrid (opt.outer_mg = 0)");
  OuterMg& g = *h->omg;
  if (k < 1 || k > g.J) throw Error(DCG_EINVAL, "level out of range");
  const int i = k - 1, nk = g.n[i];
  const int64_t len = level_len(g, k);
  switch (op) {
    case DCG_OP_OMG_APPLY:
      if (k != g.J) throw Error(DCG_EINVAL, "DCG_OP_OMG_APPLY acts on the finest level");
      omg_apply(h, in, out, st);
      break;
    case DCG_OP_OMG_LEVEL:   // out = -(0 - A*_k in)
      DCG_HIP(launch_omg_res(g.lev[i], nullptr, in, g.r[i], st));
      DCG_HIP(launch_scale(len, -1.0, g.r[i], out, st));
      break;
    case DCG_OP_OMG_RAS:
      if (k < 2) throw Error(DCG_EINVAL, "the coarsest level has no smoother");
      if (!in2) {
        DCG_HIP(launch_omg_ras(g.lev[i], in, out, true, st));
      } else {
        copy(in2, out, len, st);
        DCG_HIP(launch_omg_res(g.lev[i], in, in2, g.r[i], st));
        DCG_HIP(launch_omg_ras(g.lev[i], g.r[i], out, false, st));
      }
      break;
    case DCG_OP_OMG_RESTRICT:
      if (k < 2) throw Error(DCG_EINVAL, "restriction needs level >= 2");
      DCG_HIP(launch_omg_restrict(nk, in, out, st));
      break;
    case DCG_OP_OMG_PROLONG:
      if (k < 2) throw Error(DCG_EINVAL, "prolongation needs level >= 2");
      DCG_HIP(launch_omg_prolong(nk, in, out, true, st));
      break;
    case DCG_OP_OMG_COARSE:
      if (k != 1) throw Error(DCG_EINVAL, "the exact solve is on level 1");
      DCG_HIP(launch_omg_dense(int(len), g.cinv, in, out, st));
      break;
    case DCG_OP_OMG_WCYCLE:
      copy(in, g.f[i], len, st);
      if (in2) copy(in2, g.z[i], len, st);
      cycle(g, k, in2 ? kWarm : kZero, st);
      copy(g.z[i], out, len, st);
      break;
    default:
      throw Error(DCG_EINVAL, "unknown outer multigrid operator");
  }
}

}  // namespace dcg

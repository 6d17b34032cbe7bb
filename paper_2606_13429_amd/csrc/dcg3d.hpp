// Three-dimensional deflated CG (the d = 3 form of Section 3.1): device data
// layout and kernel launchers.
//
// Mesh: n^3 cubes of the unit cube, element e = (ez n + ey) n + ex, DG-Q1 per
// stress component, corner a = ix + 2 iy + 4 iz.  Tensor vectors hold 72
// values per element, idx = 72 e + 8 c + a with c = 3 k + i for sigma_{k+1,i+1};
// scalar vectors 8 per element, idx = 8 e + a.
//
// Face slots of an element: 0 itself, 1 / 2 the -x / +x neighbour, 3 / 4 -y /
// +y, 5 / 6 -z / +z.
//
//   At [54 + 27 12][64] the 3 x 3 block C_3 = [B_ij] of A_div (Section 3.1),
//                       row 8 j + a (test component j), column 8 i + b (trial
//                       component i within a row of the tensor), and the mass
//                       matrix of M_1, as A operands of the FP64 16 x 16 x 4
//                       MFMA: tile (r, t, h), lane l = row row_of(r, l % 16)
//                       (zero rows pad), column 8 t + 2 (l / 16) + h.  Tiles:
//                       face slots s = 1..6 (normal axis a) for t, then h, row
//                       tiles 0 and 1 where t = a, else only the one that
//                       holds the rows j = a (the other blocks are zero);
//                       then M_1 in block (t, t), the row tile that holds it;
//                       then per class c = cx + 3 cy + 9 cz (0 low side, 2 high
//                       side, 1 inside) the element's own block, t, h, r
//   Ld [7][ne][8][8]    B_11 + B_22 + B_33 (the SIPG Laplacian of
//                       Corollary 1), column-major per block
//   Dinv[ne][8][8]      inverse of the diagonal block of (dt/3) Ld,
//                       column-major (block-Jacobi preconditioner)
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dcg3 {

constexpr int kNb = 8;        // Q1 basis functions per cube
constexpr int kComp = 9;      // stress components
constexpr int kDof = 72;      // values per element of a tensor vector
constexpr int kSlots = 7;     // the element and its 6 face neighbours

constexpr int kSlotTiles = 8;                       // table tiles of a face slot
constexpr int kFixedTiles = 6 * kSlotTiles + 6;     // face slots and M_1
constexpr int kSelfTiles = 12;                      // own block of one class
constexpr int kSelfClasses = 27;
// Row of C_3 at row m of row tile r (-1: padding): a lane's results of tile 0
// are rows 4 q .. 4 q + 3, of tile 1 rows 16 + 2 q, 16 + 2 q + 1.
constexpr int row_of(int r, int m) {
  return r == 0 ? 4 * (m & 3) + (m >> 2) : ((m >> 2) < 2 ? 16 + 2 * (m & 3) + (m >> 2) : -1);
}

// Scalars of the inner PCG iteration, kept on the device between launches.
struct PcgScalars {
  double rho;       // (r, z)
  double rr;        // (r, r)
  double pq;        // (p, E p)
  double alpha, beta;
  double thresh2;   // stop once (r, r) <= thresh2
  int32_t active;   // 0 once converged: the update kernels then change nothing
  int32_t iters;    // PCG steps taken
};

// Workgroup count of the partial-sum kernels for vectors of length len.
int partial_blocks(int64_t len);

// y = A* x = inv_nu (C_9 (x) M_1) x + dt A_div x, tensor vectors; with s != NULL
// also s = Z^T y.
hipError_t launch_astar3(int n, const double* At, double inv_nu, double dt, const double* x, double* y,
                         double* s, hipStream_t st);
// q = w - dt A_div Z yh (Z = V of eq. (Vmatrix), d = 3); yh a scalar vector.
hipError_t launch_adivz3(int n, const double* At, double dt, const double* w, const double* yh,
                         double* q, hipStream_t st);
// s = Z^T w.
hipError_t launch_zt3(int64_t ne, const double* w, double* s, hipStream_t st);
// x += a Z y.
hipError_t launch_zaxpy3(int64_t ne, double a, const double* y, double* x, hipStream_t st);
// q = scale Ld p (scalar vectors) and per-workgroup partials of (p, q).
hipError_t launch_lap3(int n, const double* Ld, double scale, const double* p, double* q,
                       double* part, hipStream_t st);
// PCG set-up: r = s, x = 0, z = Dinv r, p = z, rho = (r, z), rr = (r, r),
// thresh2 = rel2 * rr, active = rr > thresh2 (two launches plus the final sums).
hipError_t launch_pcg_start(int64_t ne, const double* Dinv, const double* s, double* x, double* r,
                            double* z, double* p, double* part, PcgScalars* sc, double rel2,
                            hipStream_t st);
// One PCG step after q = E p and its partials: alpha, x += alpha p,
// r -= alpha q, z = Dinv r, rho, rr, beta, p = z + beta p.
hipError_t launch_pcg_step(int64_t ne, const double* Dinv, double* x, double* r, double* z,
                           double* p, const double* q, double* part, double* part2, int nblk_q,
                           PcgScalars* sc, hipStream_t st);
// Exact inner solve out = scale V diag(1 / (lx_i + ly_j + ly_k)) V^T in by fast
// diagonalisation (V = Vy (x) Vy (x) Vx on the tensor index (Iz, Iy, Ix);
// the y and z axes share one factor), in three launches through the scalar
// buffer t; Vd row-major [j][i] = (V_d)_{j i}, VdT its transpose.  Needs
// 2 n <= 128.
hipError_t launch_fdm_solve(int n, const double* Vx, const double* VxT, const double* Vy,
                            const double* VyT, const double* lx, const double* ly, double scale,
                            const double* in, double* out, double* t, hipStream_t st);
// out[0] = sum_i x_i y_i (fixed summation order).
hipError_t launch_dot(int64_t len, const double* x, const double* y, double* part, double* out,
                      hipStream_t st);
// y += a x; y = x + b y.
hipError_t launch_axpy(int64_t len, double a, const double* x, double* y, hipStream_t st);
hipError_t launch_xpby(int64_t len, const double* x, double b, double* y, hipStream_t st);
hipError_t launch_fill(int64_t len, double v, double* x, hipStream_t st);

}  // namespace dcg3

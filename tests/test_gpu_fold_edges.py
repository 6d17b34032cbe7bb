"""The coarse cycles kept as a matrix, at the edges of their use: two handles of
different (m1, m2) on one mesh that take turns and many smoothing steps, against the
oracle's stepwise cycles, and the accuracy over the range of dt.

Bars: 1e-12 of the largest entry for each operator of the chain at the finest level,
of which a cycle has 2 m + 4 (smoothing steps, residual, restriction, coarse map,
prolongation); m = 3 gives the 1e-11 of the other sizes."""
import numpy as np
import pytest
import scipy.linalg as sla

from dcg_workloads import THREE_D
from layout import comp_to_elem, elem_to_comp
from oracle import discretisation as d
from oracle import discretisation3d as d3
from oracle import multigrid as mg
from oracle import multigrid3d as mg3
from oracle import precond as pc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402


def _close(got, ref, m):
    got = got.cpu().numpy()
    assert np.abs(got - ref).max() <= (2 * m + 4) * 1e-12 * np.abs(ref).max()


def test_two_handles_of_one_mesh_take_turns():
    n, M = 64, 4 * 64 * 64
    H = mg.Hierarchy(d.sipg_laplacian(n), n)
    steps = [(2, 2), (1, 3), (0, 16)]
    solvers = [dcg.Solver(n, 1e-3, prec="fp64", pre=a, post=b) for a, b in steps[:2]]
    f = np.random.default_rng(5).standard_normal(M)
    ref = [mg.wcycle(H, f, np.zeros(M), H.J, a, b) for a, b in steps]
    fd = torch.from_numpy(f).cuda()
    out = torch.empty_like(fd)

    def check(i):
        print("two handles: m1, m2 = %d, %d" % steps[i], flush=True)
        out.fill_(float("nan"))
        solvers[i].apply(lib.DCG_OP_WCYCLE, fd, out, level=H.J)
        _close(out, ref[i], max(steps[i]))

    for i in (0, 1, 0, 1):
        check(i)
    solvers.append(dcg.Solver(n, 1e-3, prec="fp64", pre=0, post=16))   # the context keeps this one's now
    for i in (0, 2, 1):
        check(i)
    solvers[1].close()
    solvers[2].close()
    check(0)
    solvers[1] = dcg.Solver(n, 1e-3, prec="fp64", pre=1, post=3)       # made again
    check(1)
    solvers[1].close()
    solvers[0].close()


class _Exact:
    """The W-cycle on an oracle hierarchy in extended precision: level operators by
    exact Galerkin products, local inverses by Newton steps, the coarsest solve by
    refinement."""
    L = np.longdouble

    def __init__(self, H):
        self.J, self.A, self.P, self.S = H.J, {H.J: H.A[H.J].astype(self.L)}, {}, {}
        for k in range(H.J, 1, -1):
            self.P[k] = H.P[k].astype(self.L)
            self.A[k - 1] = (self.P[k].T @ self.A[k] @ self.P[k]).tocsr()
            self.S[k] = []
            for idx, w, inv in H.S[k].groups:
                local = np.stack([H.A[k][i][:, i].toarray() for i in idx])
                distinct, first, back = np.unique(local.reshape(len(idx), -1), axis=0, return_index=True,
                                                  return_inverse=True)
                X, B = inv[first].astype(self.L), local[first].astype(self.L)
                for _ in range(2):
                    X = X + np.matmul(X, np.eye(B.shape[-1], dtype=self.L) - np.matmul(B, X))
                self.S[k].append((idx, w.astype(self.L), X[back.reshape(-1)]))
        self.lu = sla.lu_factor(H.A[1].toarray())

    def smooth(self, k, f, z, m):
        for _ in range(m):
            r, u = f - self.A[k] @ z, np.zeros_like(z)
            for idx, w, X in self.S[k]:
                np.add.at(u, idx.ravel(), (w * np.matmul(X, r[idx][..., None])[..., 0]).ravel())
            z = z + u
        return z

    def cycle(self, k, f, z, m):
        if k == 1:
            for _ in range(8):
                z = z + sla.lu_solve(self.lu, (f - self.A[1] @ z).astype(np.float64)).astype(self.L)
            return z
        z = self.smooth(k, f, z, m)
        r = self.P[k].T @ (f - self.A[k] @ z)
        c = np.zeros_like(r)
        for _ in range(2 if k > 2 else 1):
            c = self.cycle(k - 1, r, c, m)
        return self.smooth(k, f, z + self.P[k] @ c, m)


_OMG = (lib.DCG_OP_OMG_RAS, lib.DCG_OP_OMG_LEVEL, lib.DCG_OP_OMG_RESTRICT, lib.DCG_OP_OMG_PROLONG,
        lib.DCG_OP_OMG_WCYCLE)
_MG2 = (lib.DCG_OP_RAS, lib.DCG_OP_LAPLACE, lib.DCG_OP_RESTRICT, lib.DCG_OP_PROLONG, lib.DCG_OP_WCYCLE)
_MG3 = (lib.DCG3D_MG_RAS, lib.DCG3D_MG_LAPLACE, lib.DCG3D_MG_RESTRICT, lib.DCG3D_MG_PROLONG,
        lib.DCG3D_MG_WCYCLE)


def _steps(apply, ops, f, J, m):
    """The cycle at level J = 3 with the two cycles of level 2 (which run their steps);
    apply(op, level, in, out, in2)."""
    def op(o, k, x, size, x2=None):
        out = torch.full((size,), float("nan"), dtype=torch.float64, device="cuda")
        apply(o, k, x, out, x2)
        return out
    ras, level, restrict, prolong, wcycle = ops
    N, M = f.numel(), f.numel() // (8 if ops is _MG3 else 4)
    z = None
    for _ in range(m):
        z = op(ras, J, f, N, z)
    r = op(restrict, J, f - op(level, J, z, N), M)
    c = op(wcycle, J - 1, r, M)
    c = op(wcycle, J - 1, r, M, c)
    z = z + op(prolong, J, c, N)
    for _ in range(m):
        z = op(ras, J, f, N, z)
    return z


@pytest.mark.parametrize("dt,m", [(1e-6, 1), (1e-6, 40), (1e-2, 1), (0.1, 1), (1.0, 1), (1.0, 2), (1.0, 40),
                                  (100.0, 1), (100.0, 4)])
def test_outer_multigrid_matrix_is_as_accurate_as_the_steps(dt, m):
    """The error of the application against that of its steps, both from the exact cycle
    (the operator's condition, 1e5 at the ends of the range, sets its size): at most
    twice, root mean square over four right-hand sides of random rounding."""
    n = 32
    H = pc.Hierarchy(d.operator(n, dt), n)
    X = _Exact(H)
    s = dcg.Solver(n, dt, prec="fp64", outer="fcg", outer_mg=m)
    err = np.zeros((2, 4))
    for seed in range(4):
        f = np.random.default_rng(seed).standard_normal(16 * n * n)
        x = comp_to_elem(X.cycle(X.J, elem_to_comp(f, n).astype(X.L), np.zeros(f.size, dtype=X.L), m), n)
        fd = torch.from_numpy(f).cuda()
        out = torch.full_like(fd, float("nan"))
        s.apply(lib.DCG_OP_OMG_APPLY, fd, out, level=H.J)
        y = _steps(lambda o, k, x, t, w: s.apply(o, x, t, level=k, in2=w), _OMG, fd, H.J, m)
        for i, y in enumerate((out, y)):
            err[i, seed] = np.abs(y.cpu().numpy() - x).max() / np.abs(x).max()
    s.close()
    matrix, steps = np.sqrt((err ** 2).mean(axis=1))
    print("outer mg n=%d dt=%g m=%d: matrix %.1e steps %.1e" % (n, dt, m, matrix, steps), flush=True)
    assert matrix <= 2 * steps


def test_3d_many_smoothing_steps():
    n, m = 16, 40
    print("3d mg n=%d m=%d" % (n, m), flush=True)
    s = dcg.Solver3D(n, 1e-3, nu=THREE_D["nu"], penalty=THREE_D["penalty"], inner="mg", smooth=m)
    J, c = s.mg_levels()
    H = mg3.Hierarchy(d3.sipg_laplacian(n, THREE_D["penalty"]), n, coarsest=c)
    f = np.random.default_rng(m).standard_normal(8 * n ** 3)
    fd = torch.from_numpy(f).cuda()
    out = torch.full_like(fd, float("nan"))
    s.mg_apply(lib.DCG3D_MG_WCYCLE, J, fd, out)
    _close(out, mg.wcycle(H, f, np.zeros_like(f), J, m, m), m)
    s.close()


@pytest.mark.parametrize("penalty,m", [(10.0, 1), (10.0, 2), (1e4, 2), (1e6, 2)])
def test_2d_matrix_is_as_accurate_as_the_steps(penalty, m):
    """The same for the inner multigrid (levels of 64, 32 and 16 squares), single and
    batched; a penalty of 1e4 and more makes the Laplacian ill-conditioned."""
    n, M = 64, 4 * 64 * 64
    H = mg.Hierarchy(d.sipg_laplacian(n, penalty), n)
    X = _Exact(H)
    s = dcg.Solver(n, 1e-3, prec="fp64", penalty=penalty, pre=m, post=m)
    zero = torch.zeros(M, dtype=torch.float64, device="cuda")

    def apply(o, k, x, t, w):
        s.apply(o, x, t, level=k, in2=zero if o == lib.DCG_OP_RAS and w is None else w)
    err = np.zeros((3, 4))
    f = np.random.default_rng(3).standard_normal((16, M))
    fb = torch.from_numpy(np.ascontiguousarray(f.reshape(16, n * n, 4).transpose(1, 0, 2)).reshape(-1)).cuda()
    zb = torch.full_like(fb, float("nan"))
    s.apply(lib.DCG_OP_WCYCLE_BATCH, fb, zb, level=3)
    zb = zb.cpu().numpy().reshape(n * n, 16, 4)
    for c in range(4):
        x = X.cycle(3, f[c].astype(X.L), np.zeros(M, dtype=X.L), m)
        fd = torch.from_numpy(f[c].copy()).cuda()
        out = torch.full_like(fd, float("nan"))
        s.apply(lib.DCG_OP_WCYCLE, fd, out, level=3)
        y = _steps(apply, _MG2, fd, 3, m)
        for i, v in enumerate((out.cpu().numpy(), zb[:, c].reshape(-1), y.cpu().numpy())):
            err[i, c] = np.abs(v - x).max() / np.abs(x).max()
    s.close()
    matrix, batch, steps = np.sqrt((err ** 2).mean(axis=1))
    print("2d n=%d penalty=%g m=%d: matrix %.1e batch %.1e steps %.1e" % (n, penalty, m, matrix, batch, steps),
          flush=True)
    assert max(matrix, batch) <= 2 * steps


@pytest.mark.parametrize("penalty,m", [(40.0, 1), (40.0, 3), (1e5, 3)])
def test_3d_matrix_is_as_accurate_as_the_steps(penalty, m):
    """The same for the 3D inner multigrid (levels of 16, 8 and 4 cubes)."""
    n = 16
    H = mg3.Hierarchy(d3.sipg_laplacian(n, penalty), n, coarsest=4)
    X = _Exact(H)
    s = dcg.Solver3D(n, 1e-3, penalty=penalty, inner="mg", levels=3, smooth=m)
    err = np.zeros((2, 4))
    for seed in range(4):
        f = np.random.default_rng(seed).standard_normal(8 * n ** 3)
        x = X.cycle(3, f.astype(X.L), np.zeros(f.size, dtype=X.L), m)
        fd = torch.from_numpy(f).cuda()
        out = torch.full_like(fd, float("nan"))
        s.mg_apply(lib.DCG3D_MG_WCYCLE, 3, fd, out)
        y = _steps(lambda o, k, x, t, w: s.mg_apply(o, k, x, t, w), _MG3, fd, 3, m)
        for i, y in enumerate((out, y)):
            err[i, seed] = np.abs(y.cpu().numpy() - x).max() / np.abs(x).max()
    s.close()
    matrix, steps = np.sqrt((err ** 2).mean(axis=1))
    print("3d n=%d penalty=%g m=%d: matrix %.1e steps %.1e" % (n, penalty, m, matrix, steps), flush=True)
    assert matrix <= 2 * steps


def test_server_groups_give_the_matrix_back_and_go_on():
    """Two running groups of a 2 GiB server give their matrices back when a third needs
    the room (FP64, n = 64, 128 and 256 hold 0.12 + 0.38 + 1.43 GiB), go on with the steps
    and serve further requests: every solution within 1e-8 of the single solver's."""
    budget, dt = 2 << 30, 1e-4
    need = [lib.dcg_server_group_bytes(dcg.Server.mesh(n), lib.DCG_FP64) for n in (64, 128, 256)]
    assert sum(need) <= budget < sum(need) + (1 << 27)
    ref, bs = {}, {}
    for n in (64, 128, 256):
        bs[n] = torch.from_numpy(np.random.default_rng(n).standard_normal(16 * n * n)).cuda()
        ref[n] = torch.empty_like(bs[n])
        s = dcg.Solver(n, dt, prec="fp64")
        status, _ = s.solve(bs[n], ref[n], tol=1e-8)
        s.close()
        assert status == lib.DCG_OK
    srv = dcg.Server(prec="fp64", hbm_budget_bytes=budget)
    for mix in ((64, 128, 256), (64, 64, 128), (256, 64)):
        print("server mix", mix, flush=True)
        xs = [torch.full_like(bs[n], float("nan")) for n in mix]
        torch.cuda.synchronize()
        tickets = [srv.submit(n, dt, bs[n], x, tol=1e-8) for n, x in zip(mix, xs)]
        for n, x, t in zip(mix, xs, tickets):
            status, _ = srv.wait(t, timeout=100)
            assert status == lib.DCG_OK
            assert float((x - ref[n]).norm()) <= 1e-8 * float(ref[n].norm()), n
    srv.close()

"""Restriction of the residual by 16 x 16 tiles (levels from 64 x 64) and the
refinement residual by one thread per square: one level below the finest solved
exactly (levels = 2), no pre-smoothing, so that the cycle is restriction, exact
coarse solve, prolongation and one step; from zero and from an iterate.

Bars: the cycle's at these sizes, 16 eps n^2 of the largest entry; the inner solve
by its residual against its own tolerance, c_F 1e-8 with c_F <= 1."""
import numpy as np
import pytest

from oracle import discretisation as d
from oracle import multigrid as mg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("n", [32, 64, 128])
@pytest.mark.parametrize("m1", [0, 1])
def test_two_level_cycle(n, prec, m1):
    print("two-level cycle n=%d m1=%d %s" % (n, m1, prec), flush=True)
    H = mg.Hierarchy(d.sipg_laplacian(n), n)
    real = torch.float32 if prec == "mixed" else torch.float64
    rng = np.random.default_rng(n + m1)
    fd = torch.from_numpy(rng.standard_normal(4 * n * n)).to("cuda", real)
    zd = torch.from_numpy(rng.standard_normal(4 * n * n) * 1e-3).to("cuda", real)
    f, z0 = fd.double().cpu().numpy(), zd.double().cpu().numpy()
    s = dcg.Solver(n, 1e-3, prec=prec, levels=2, pre=m1, post=1)
    out = torch.full_like(fd, float("nan"))
    for start in (None, zd):
        s.apply(lib.DCG_OP_WCYCLE, fd, out, level=2, **({} if start is None else {"in2": start}))
        z = np.zeros_like(f) if start is None else z0.copy()
        J = H.J
        for _ in range(m1):
            z = z + H.S[J].apply(f - H.A[J] @ z)
        rc = H.P[J].T @ (f - H.A[J] @ z)
        z = z + H.P[J] @ _solve(H.A[J - 1], rc)
        z = z + H.S[J].apply(f - H.A[J] @ z)
        got = out.double().cpu().numpy()
        assert np.abs(got - z).max() <= 16 * float(torch.finfo(real).eps) * n * n * np.abs(z).max()
    s.close()


def _solve(A, b):
    import scipy.sparse.linalg as sl
    return sl.spsolve(A.tocsc(), b)


@pytest.mark.parametrize("n", [16, 32, 64, 128])
def test_refined_inner_residual(n):
    print("refined inner solve n=%d" % n, flush=True)
    s = dcg.Solver(n, 1e-3, prec="mixed")
    b = torch.from_numpy(np.random.default_rng(n).standard_normal(4 * n * n)).cuda()
    y = torch.full_like(b, float("nan"))
    s.apply(lib.DCG_OP_INNER, b, y)
    s.close()
    r = b.cpu().numpy() - (1e-3 / 2) * (d.sipg_laplacian(n) @ y.cpu().numpy())
    assert np.linalg.norm(r) <= 1e-8 * np.linalg.norm(b.cpu().numpy())

"""A* and A_div Z from the operator tables at the edges of their launches:
n = 16 (one wavefront holds two rows of squares and up to five classes), 32
(a wavefront is one row, three classes) and 128 (the deflation kernel runs one
trip per workgroup, larger meshes several).  Bar: 1e-13 of the largest entry of
|A*| |x| (at most 80 FP64 terms a row)."""
import numpy as np
import pytest

from layout import comp_to_elem, elem_to_comp
from oracle import discretisation as d2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402


@pytest.mark.parametrize("n", [16, 32, 128])
def test_astar_and_adivz(n):
    print("operator tables n=%d" % n, flush=True)
    dt, nu = 3e-2, 0.7
    s = dcg.Solver(n, dt, nu=nu, prec="fp64")
    rng = np.random.default_rng(n)
    x, y = rng.standard_normal(16 * n * n), rng.standard_normal(4 * n * n)
    A, V = d2.operator(n, dt, nu, 10.0), d2.deflation_basis(n)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    out = torch.full_like(xd, float("nan"))
    s.apply(lib.DCG_OP_ASTAR, xd, out)
    bar = 1e-13 * (abs(A) @ np.abs(elem_to_comp(x, n))).max()
    assert np.abs(out.cpu().numpy() - comp_to_elem(A @ elem_to_comp(x, n), n)).max() <= bar
    s.apply(lib.DCG_OP_ADIVZ, yd, out)
    bar = 1e-13 * (abs(A) @ np.abs(V @ y)).max()          # dt A_div Z y = A* Z y
    assert np.abs(dt * out.cpu().numpy() - comp_to_elem(A @ (V @ y), n)).max() <= bar
    s.close()

"""The 3D A* product, A_div Z and the exact inner solve at the sizes where
their tilings end: 16 elements per wavefront (ragged last group, several
classes of elements in one), one or two groups per workgroup (from 512 groups,
n >= 21), 16-row tiles and steps of 8 of the fast diagonalisation.

Bars: the operators 1e-13 of the largest entry of |A*| |x| (at most 170 terms
summed in FP64); the exact inner solve by its residual, 1e-11 as at the other
sizes."""
import numpy as np
import pytest

from layout import comp_to_elem3, elem_to_comp3
from oracle import discretisation3d as d3

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402


@pytest.mark.parametrize("n", [4, 7, 9, 21])
def test_astar_adivz_inner_at_tile_edges(n):
    print("3d mfma operators n=%d" % n, flush=True)
    dt, nu, pen = 3e-2, 0.7, 40.0
    s = dcg.Solver3D(n, dt, nu=nu, penalty=pen)
    rng = np.random.default_rng(n)
    m = 8 * n ** 3
    x, y = rng.standard_normal(9 * m), rng.standard_normal(m)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    out, sc = torch.full_like(xd, float("nan")), torch.full_like(yd, float("nan"))
    As = d3.operator(n, dt, nu=nu, penalty=pen)
    bar = 1e-13 * (abs(As) @ np.abs(elem_to_comp3(x, n))).max()
    s.apply(lib.DCG3D_OP_ASTAR, xd, out)
    assert np.abs(out.cpu().numpy() - comp_to_elem3(As @ elem_to_comp3(x, n), n)).max() <= bar
    V = d3.deflation_basis(n)
    ref = As @ (V @ y)                       # dt A_div Z y: M Z = 0
    bar = 1e-13 * (abs(As) @ np.abs(V @ y)).max()
    s.apply(lib.DCG3D_OP_ADIVZ, yd, out)
    assert np.abs(dt * out.cpu().numpy() - comp_to_elem3(ref, n)).max() <= bar
    s.apply(lib.DCG3D_OP_INNER, yd, sc, 1e-12)
    z = sc.cpu().numpy()
    assert np.linalg.norm(V.T @ (As @ (V @ z)) - y) <= 1e-11 * np.linalg.norm(y)
    s.close()

"""The outer multigrid at n = 32: the finest level is the smallest that runs as
tasks of 16 squares (ragged tasks in most classes) and the level of 16 x 16 squares
is kept as a matrix, for one, two and three smoothing steps (every branch of the
powers it is formed from).  Bars as at the other sizes: 1e-12 of the largest entry
for one operator, 1e-11 for the W-cycle."""
import numpy as np
import pytest

from layout import comp_to_elem, elem_to_comp
from oracle import discretisation as d
from oracle import multigrid as mg
from oracle import precond as pc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402


def _close(got, ref, rel):
    assert np.abs(got.cpu().numpy() - ref).max() <= rel * np.abs(ref).max()


@pytest.mark.parametrize("m", [1, 2, 3])
def test_tasks_and_folded_level(m):
    n, dt = 32, 3e-3
    print("outer mg tasks n=%d m=%d" % (n, m), flush=True)
    H = pc.Hierarchy(d.operator(n, dt), n)
    s = dcg.Solver(n, dt, prec="fp64", outer="fcg", outer_mg=m)
    J = H.J
    rng = np.random.default_rng(m)
    f, z = rng.standard_normal(16 * n * n), rng.standard_normal(16 * n * n)
    fd, zd = torch.from_numpy(f).cuda(), torch.from_numpy(z).cuda()
    fc, zc = elem_to_comp(f, n), elem_to_comp(z, n)
    out = torch.full_like(fd, float("nan"))
    s.apply(lib.DCG_OP_OMG_LEVEL, zd, out, level=J)
    _close(out, comp_to_elem(H.A[J] @ zc, n), 1e-12)
    s.apply(lib.DCG_OP_OMG_RAS, fd, out, level=J, in2=zd)
    _close(out, comp_to_elem(zc + H.S[J].apply(fc - H.A[J] @ zc), n), 1e-12)
    s.apply(lib.DCG_OP_OMG_WCYCLE, fd, out, level=J, in2=zd)
    _close(out, comp_to_elem(mg.wcycle(H, fc, zc, J, m, m), n), 1e-11)
    for _ in range(2):                     # the captured application, replayed
        s.apply(lib.DCG_OP_OMG_APPLY, fd, out, level=J)
        _close(out, comp_to_elem(mg.wcycle(H, fc, np.zeros_like(fc), J, m, m), n), 1e-11)
    s.close()

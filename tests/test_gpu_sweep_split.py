"""The grouped RAS step by its number of workgroups (n = 128): 4 x 4 tiles per group
split over two workgroups, 2 x 2 tiles with 8 wavefronts, single tiles with 4; and
n = 64, split over four, the choice made without ras_group.  The step from an
iterate, and the W-cycle, whose first post-smoothing step adds the prolongated
correction.

Bars of the same step and cycle at these sizes: step 2e-4 / 1e-12 of the largest
entry, cycle 16 eps n^2."""
import numpy as np
import pytest

from oracle import discretisation as d
from oracle import multigrid as mg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402

_H = {}


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("n,group", [(128, 4), (128, 2), (128, 1), (64, 0)])
def test_step_and_cycle_of_each_split(n, group, prec):
    print("split n=%d group=%d %s" % (n, group, prec), flush=True)
    if n not in _H:
        _H[n] = mg.Hierarchy(d.sipg_laplacian(n), n)
    H = _H[n]
    real = torch.float32 if prec == "mixed" else torch.float64
    eps = float(torch.finfo(real).eps)
    rng = np.random.default_rng(n + group)
    fd = torch.from_numpy(rng.standard_normal(4 * n * n)).to("cuda", real)
    zd = torch.from_numpy(rng.standard_normal(4 * n * n) * 1e-3).to("cuda", real)
    f, z = fd.double().cpu().numpy(), zd.double().cpu().numpy()
    s = dcg.Solver(n, 1e-3, prec=prec, ras_group=group)
    out = torch.full_like(fd, float("nan"))
    s.apply(lib.DCG_OP_RAS, fd, out, level=H.J, in2=zd)
    ref = z + H.S[H.J].apply(f - H.A[H.J] @ z)
    assert np.abs(out.double().cpu().numpy() - ref).max() <= (2e-4 if prec == "mixed" else 1e-12) * np.abs(ref).max()
    out.fill_(float("nan"))
    s.apply(lib.DCG_OP_WCYCLE, fd, out, level=H.J)
    s.close()
    ref = mg.wcycle(H, f, np.zeros_like(f), H.J)
    assert np.abs(out.double().cpu().numpy() - ref).max() <= 16 * eps * n * n * np.abs(ref).max()

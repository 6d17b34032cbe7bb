"""The fast-diagonalisation solve of small grids, N = 2 n in {32, 64, 128} in two
passes and 256 in four products: the exact inner solve, and the coarsest solve in
both level types.

Bars: the inner solve by its residual, 40 n^2 eps (the condition number of the
SIPG Laplacian times the unit round-off); the FP32 coarsest solve against the
FP64 one, 2^-23 of the largest entry (the input is representable, the output is
rounded once)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402


@pytest.mark.parametrize("n", [16, 32, 64, 128])
def test_small_exact_inner_residual(n):
    print("exact inner residual n=%d" % n, flush=True)
    s = dcg.Solver(n, 1e-3, inner="exact")
    rhs = torch.from_numpy(np.random.default_rng(n).standard_normal(4 * n * n)).cuda()
    y, back = torch.full_like(rhs, float("nan")), torch.empty_like(rhs)
    v, w = (torch.empty(16 * n * n, dtype=torch.float64, device="cuda") for _ in range(2))
    s.apply(lib.DCG_OP_INNER, rhs, y)
    s.apply(lib.DCG_OP_Z, y, v)
    s.apply(lib.DCG_OP_ASTAR, v, w)
    s.apply(lib.DCG_OP_ZT, w, back)          # E y = Z^T A* Z y
    s.close()
    assert float((back - rhs).norm()) <= 40 * n * n * 2.0 ** -53 * float(rhs.norm())


@pytest.mark.parametrize("n", [32, 64, 128])
def test_small_coarsest_solve_in_fp32_equals_fp64(n):
    print("coarsest solve n=%d" % n, flush=True)
    f = torch.from_numpy(np.random.default_rng(n).standard_normal(4 * n * n).astype(np.float32)).cuda()
    z32, z64 = torch.empty_like(f), torch.empty_like(f, dtype=torch.float64)
    for prec, fin, out in (("mixed", f, z32), ("fp64", f.double(), z64)):
        s = dcg.Solver(n, 1e-3, prec=prec, levels=1)
        s.apply(lib.DCG_OP_COARSE, fin, out, level=1)
        s.close()
    assert float((z32.double() - z64).abs().max()) <= 2.0 ** -23 * float(z64.abs().max())

"""Vectors that start at an odd element of their storage: every entry point takes
contiguous slices, which are aligned to their elements only, and the kernels read
and write them 16 bytes at a time.  Each call on such slices against the same call on
aligned buffers: the same kernels in the same order, so the outputs are equal bit
for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lib = pytest.importorskip("paper_2606_13429_amd._binding")
import paper_2606_13429_amd as dcg  # noqa: E402


def _vec(a, shift):
    """A device copy of ``a`` that starts at element ``shift`` of its storage."""
    buf = torch.zeros(a.size + shift, dtype=torch.from_numpy(a[:1]).dtype, device="cuda")
    v = buf[shift:]
    v.copy_(torch.from_numpy(a))
    assert v.is_contiguous() and v.data_ptr() % 16 == (shift * a.itemsize) % 16
    return v


def _both(call, inp, nout, dtype=np.float64, in2=None):
    """call(in, out[, in2]) on aligned and on shifted vectors."""
    got = []
    for shift in (0, 1):
        out = _vec(np.full(nout, np.nan, dtype=dtype), shift)
        args = (_vec(inp, shift), out) + (() if in2 is None else (_vec(in2, shift),))
        call(*args)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    assert np.isfinite(got[0]).all() and np.any(got[0])
    assert np.array_equal(got[0], got[1])


def _rand(n, seed, dtype=np.float64):
    return np.random.default_rng(seed).standard_normal(n).astype(dtype)


@pytest.mark.parametrize("n,inner", [(16, "mg"), (64, "mg"), (128, "exact")])
def test_operators(n, inner):
    s = dcg.Solver(n, 1e-3, inner=inner)
    N, M = 16 * n * n, 4 * n * n
    for op, m, k in ((lib.DCG_OP_ASTAR, N, N), (lib.DCG_OP_ZT, N, M), (lib.DCG_OP_Z, M, N),
                     (lib.DCG_OP_ADIVZ, M, N), (lib.DCG_OP_INNER, M, M), (lib.DCG_OP_DEFLATED, N, N)):
        print("n=%d %s op=%d" % (n, inner, op), flush=True)
        _both(lambda i, o: s.apply(op, i, o), _rand(m, op), k)
    print("n=%d %s solve" % (n, inner), flush=True)
    _both(lambda b, x: s.solve(b, x), _rand(N, 9), N)
    s.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("group", [-1, 0])
def test_level_operators(prec, group):
    n = 64
    dt = np.float64 if prec == "fp64" else np.float32
    s = dcg.Solver(n, 1e-3, prec=prec, ras_group=group)
    for k in (2, 3):
        M = 4 * (n >> (3 - k)) ** 2
        f, z = _rand(M, 1, dt), _rand(M, 2, dt)
        print("level %d %s" % (k, prec), flush=True)
        _both(lambda i, o: s.apply(lib.DCG_OP_LAPLACE, i, o, level=k), f, M, dt)
        _both(lambda i, o, w: s.apply(lib.DCG_OP_RAS, i, o, level=k, in2=w), f, M, dt, z)
        _both(lambda i, o: s.apply(lib.DCG_OP_RESTRICT, i, o, level=k), f, M // 4, dt)
        _both(lambda i, o: s.apply(lib.DCG_OP_PROLONG, i, o, level=k), f[:M // 4].copy(), M, dt)
        _both(lambda i, o: s.apply(lib.DCG_OP_WCYCLE, i, o, level=k), f, M, dt)
        fb, zb = _rand(16 * M, 3, dt), _rand(16 * M, 4, dt)
        _both(lambda i, o, w: s.apply(lib.DCG_OP_RAS_BATCH, i, o, level=k, in2=w), fb, 16 * M, dt, zb)
        _both(lambda i, o: s.apply(lib.DCG_OP_WCYCLE_BATCH, i, o, level=k), fb, 16 * M, dt)
    _both(lambda i, o: s.apply(lib.DCG_OP_COARSE, i, o, level=1), _rand(1024, 4, dt), 1024, dt)
    s.close()


def test_outer_multigrid():
    n = 64
    s = dcg.Solver(n, 1e-3, outer="fcg", outer_mg=2, inner="exact")
    for k in (2, 3, 4):
        N = 16 * (n >> (4 - k)) ** 2
        r, z = _rand(N, k), _rand(N, 10 + k)
        print("outer level %d" % k, flush=True)
        for op in (lib.DCG_OP_OMG_LEVEL, lib.DCG_OP_OMG_RAS, lib.DCG_OP_OMG_WCYCLE):
            _both(lambda i, o: s.apply(op, i, o, level=k), r, N)
        _both(lambda i, o, w: s.apply(lib.DCG_OP_OMG_RAS, i, o, level=k, in2=w), r, N, in2=z)
    _both(lambda i, o: s.apply(lib.DCG_OP_OMG_COARSE, i, o, level=1), _rand(1024, 3), 1024)
    _both(lambda i, o: s.apply(lib.DCG_OP_OMG_APPLY, i, o, level=4), _rand(16 * n * n, 5), 16 * n * n)
    s.close()


@pytest.mark.parametrize("n,inner", [(5, "exact"), (16, "mg")])
def test_3d(n, inner):
    s = dcg.Solver3D(n, 1e-3, inner=inner)
    N, M = 72 * n ** 3, 8 * n ** 3
    for op, m, k in ((lib.DCG3D_OP_ASTAR, N, N), (lib.DCG3D_OP_ADIVZ, M, N), (lib.DCG3D_OP_INNER, M, M),
                     (lib.DCG3D_OP_DEFLATED, N, N), (lib.DCG3D_OP_REDUCED, M, M)):
        print("3d n=%d %s op=%d" % (n, inner, op), flush=True)
        _both(lambda i, o: s.apply(op, i, o, tol=1e-8), _rand(m, op), k)
    if inner == "mg":
        J, _ = s.mg_levels()
        for k in range(2, J + 1):
            L = 8 * (n >> (J - k)) ** 3
            f, z = _rand(L, k), _rand(L, 10 + k)
            print("3d level %d" % k, flush=True)
            for op in (lib.DCG3D_MG_LAPLACE, lib.DCG3D_MG_RAS, lib.DCG3D_MG_WCYCLE):
                _both(lambda i, o: s.mg_apply(op, k, i, o), f, L)
            _both(lambda i, o, w: s.mg_apply(lib.DCG3D_MG_RAS, k, i, o, in2=w), f, L, in2=z)
    else:
        print("3d n=%d %s solve" % (n, inner), flush=True)
        _both(lambda b, x: s.solve(b, x), _rand(N, 9), N)
    s.close()

"""Workloads of the solver as a program calls them: the operators of the
deflated CG through ``dcg_apply`` / ``dcg3d_apply``, and whole solves.

``listed()`` names the cases, ``draw(rng)`` gives another case of the same
ranges, ``prepare`` makes the device inputs and the handle, ``run`` is one
pass through the public entry points, ``work`` the bytes and operations a pass
cannot do without, and ``exact`` the result in FP64 from the definitions of
the discretisation: the uniform grid's forms are sums of Kronecker products of
one-dimensional DG-Q1 matrices, applied here as dense torch products.
"""
import math

import torch

import paper_2606_13429_amd as dcg

TOL = 1e-8        # outer tolerance of every workload
C_F = 0.01        # fixed inner tolerance factor: c_F * TOL


# ------------------------------------------------------------------- cases
def listed():
    return [
        # smallest workload of the repository (16 x 16 squares, FP64): one A* product, where the
        # call's own latency counts
        dict(name="astar2d_n16", kind="astar2d", n=16, dt=1e-2),
        # the operator of the BDF2 time stepping on its 1024 x 1024 mesh (alpha = 2 dt / 3)
        dict(name="astar2d_n1024", kind="astar2d", n=1024, dt=2e-5 / 3.0),
        # one outer iteration's operator M_D in the FP64 dt sweep, default (full) hierarchy
        dict(name="deflated2d_n128_fp64", kind="deflated2d", n=128, dt=1e-3, prec="fp64", levels=0, pre=2,
             post=2),
        # the same at the headline size: mixed form, four multigrid levels
        dict(name="deflated2d_n512_mixed", kind="deflated2d", n=512, dt=1e-4, prec="mixed", levels=4, pre=2,
             post=2),
        # the serving engine's W-cycle over a full batch of 16 requests, FP64 form (one FP32 cycle
        # alone leaves 3e-3 of rounding in its output, which the mixed form's FP64 refinement takes
        # out: that form is measured by the solves)
        dict(name="wcycle_batch_n128", kind="wcycle_batch", n=128, pre=2, post=2),
        # the exact inner solve of the exact-inner deflated CG at the headline size
        dict(name="inner_exact_n512", kind="inner_exact", n=512, dt=1e-4),
        # the multigrid preconditioner on A* (one application per outer iteration)
        dict(name="outer_mg_n256", kind="outer_mg", n=256, dt=1e-4, m=4),
        # 3D, one outer iteration's operator with the exact inner solve: the 3D workload's mesh
        dict(name="deflated3d_n32", kind="deflated3d", n=32, dt=1e-3),
        # and a small mesh with an odd number of cubes per side
        dict(name="deflated3d_n13", kind="deflated3d", n=13, dt=1e-2),
        # 3D multigrid inner solve: one W-cycle, 10 pre- and post-smoothing steps
        dict(name="wcycle3d_n32", kind="wcycle3d", n=32, smooth=10),
        # a whole solve at the headline size and a time step of the time-stepping workload
        dict(name="solve2d_n512", kind="solve2d", n=512, dt=1e-5, prec="mixed", levels=4),
        # serving: a burst of 16 requests on one of the smaller served meshes, dt over the trace's
        # range up to where its requests converge in some hundred iterations
        dict(name="serve_n64", kind="serve", n=64, count=16, lo=-6.0, hi=-3.0, prec="mixed"),
    ]


def _log(rng, lo, hi):
    return 10.0 ** rng.uniform(lo, hi)


def draw(rng):
    kind = rng.choice(["astar2d", "deflated2d", "wcycle_batch", "inner_exact", "outer_mg", "deflated3d",
                       "wcycle3d", "solve2d", "serve"])
    if kind == "astar2d":
        return dict(kind=kind, n=rng.choice([16, 32, 64, 128, 256, 512]), dt=_log(rng, -6, -1))
    if kind == "deflated2d":
        n = rng.choice([16, 32, 64, 128, 256, 512])
        levels = rng.choice([0, 0, 3, 4])
        if levels and n >> (levels - 1) < 16:
            levels = 0
        m = rng.choice([1, 2, 2, 2, 5])
        return dict(kind=kind, n=n, dt=_log(rng, -6, -1), prec=rng.choice(["fp64", "mixed"]), levels=levels,
                    pre=m, post=m)
    if kind == "wcycle_batch":
        m = rng.choice([1, 2, 2, 3])
        return dict(kind=kind, n=rng.choice([32, 64, 128, 256]), pre=m, post=m, dt=_log(rng, -6, -1))
    if kind == "inner_exact":
        return dict(kind=kind, n=rng.choice([16, 32, 64, 128, 256, 512]), dt=_log(rng, -6, -1))
    if kind == "outer_mg":
        return dict(kind=kind, n=rng.choice([32, 64, 128, 256]), dt=_log(rng, -5, -2), m=rng.randint(1, 6))
    if kind == "deflated3d":
        return dict(kind=kind, n=round(math.exp(rng.uniform(math.log(2), math.log(32)))), dt=_log(rng, -5, 0))
    if kind == "wcycle3d":
        return dict(kind=kind, n=rng.choice([4, 6, 8, 12, 16, 24, 32]), smooth=rng.randint(2, 10))
    if kind == "solve2d":
        n = rng.choice([16, 32, 64, 128, 256])
        return dict(kind=kind, n=n, dt=_log(rng, -6, 2 * math.log10(1.2 / n)), prec=rng.choice(["fp64", "mixed"]),
                    levels=4 if n >= 128 else 0)
    return dict(kind=kind, n=rng.choice([16, 32, 64, 128]), count=rng.randint(3, 16), lo=-6.0,
                hi=round(rng.uniform(-5.0, -3.5), 2), prec=rng.choice(["fp64", "mixed"]))


def _dts(case):
    """Time steps of a serving burst, evenly spread over the exponents [lo, hi]."""
    c = case["count"]
    return [10.0 ** (case["lo"] + (case["hi"] - case["lo"]) * i / max(1, c - 1)) for i in range(c)]


NU3, PENALTY3 = 0.5, 40.0     # viscosity and penalty of the 3D workload


# ------------------------------------------------------------------- a pass
def _randn(count, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(count, dtype=torch.float64, device="cuda", generator=g)


def prepare(case, seed):
    k, n = case["kind"], case["n"]
    if k == "astar2d":
        x = _randn(16 * n * n, seed)
        return dict(case=case, s=dcg.Solver(n, case["dt"], prec="fp64"), x=x, out=torch.empty_like(x))
    if k == "deflated2d":
        x = _randn(16 * n * n, seed)
        s = dcg.Solver(n, case["dt"], prec=case["prec"], levels=case["levels"], pre=case["pre"],
                       post=case["post"])
        return dict(case=case, s=s, x=x, out=torch.empty_like(x))
    if k == "wcycle_batch":
        x = _randn(16 * 4 * n * n, seed)
        s = dcg.Solver(n, case.get("dt", 1e-3), prec="fp64", pre=case["pre"], post=case["post"])
        return dict(case=case, s=s, x=x, out=torch.empty_like(x), level=dcg.dcg_num_levels(n))
    if k == "inner_exact":
        x = _randn(4 * n * n, seed)
        return dict(case=case, s=dcg.Solver(n, case["dt"], inner="exact"), x=x, out=torch.empty_like(x))
    if k == "outer_mg":
        x = _randn(16 * n * n, seed)
        s = dcg.Solver(n, case["dt"], outer="fcg", outer_mg=case["m"])
        return dict(case=case, s=s, x=x, out=torch.empty_like(x), level=int(math.log2(n // 8)) + 1)
    if k == "deflated3d":
        x = _randn(72 * n ** 3, seed)
        s = dcg.Solver3D(n, case["dt"], nu=NU3, penalty=PENALTY3)
        return dict(case=case, s=s, x=x, out=torch.empty_like(x))
    if k == "wcycle3d":
        x = _randn(8 * n ** 3, seed)
        s = dcg.Solver3D(n, 1e-3, nu=NU3, penalty=PENALTY3, inner="mg", smooth=case["smooth"])
        return dict(case=case, s=s, x=x, out=torch.empty_like(x), level=s.mg_levels()[0])
    if k == "solve2d":
        x = _randn(16 * n * n, seed)
        return dict(case=case, s=dcg.Solver(n, case["dt"], prec=case["prec"], levels=case["levels"]), x=x,
                    out=torch.empty_like(x))
    if k == "serve":
        x = _randn(case["count"] * 16 * n * n, seed).view(case["count"], -1)
        s = dcg.Server(prec=case["prec"])
        s.prepare(n)
        return dict(case=case, s=s, x=x, out=torch.empty_like(x), dts=_dts(case))
    raise ValueError(k)


def run(state):
    k, s, x, out = state["case"]["kind"], state["s"], state["x"], state["out"]
    if k == "astar2d":
        s.apply(dcg.DCG_OP_ASTAR, x, out)
    elif k == "deflated2d":
        s.apply(dcg.DCG_OP_DEFLATED, x, out)
    elif k == "wcycle_batch":
        s.apply(dcg.DCG_OP_WCYCLE_BATCH, x, out, level=state["level"])
    elif k == "inner_exact":
        s.apply(dcg.DCG_OP_INNER, x, out)
    elif k == "outer_mg":
        s.apply(dcg.DCG_OP_OMG_APPLY, x, out, level=state["level"])
    elif k == "deflated3d":
        s.apply(dcg.DCG3D_OP_DEFLATED, x, out, tol=C_F * TOL)
    elif k == "wcycle3d":
        s.mg_apply(dcg.DCG3D_MG_WCYCLE, state["level"], x, out)
    elif k == "solve2d":
        s.solve(x, out, tol=TOL)
    elif k == "serve":
        n = state["case"]["n"]
        tickets = [s.submit(n, dt, x[i], out[i], tol=TOL) for i, dt in enumerate(state["dts"])]
        for t in tickets:
            s.wait(t)
    return out


# ------------------------------------------------------------------- work
def _cycle_flops(n, pre, post):
    """One 2D W-cycle: per square and smoothing step a 128 x 128 tile solve over 16 squares and the
    residual; the levels below, a quarter of the size and visited twice, add the same once."""
    return 2.0 * n * n * ((pre + post) * (2.0 * 128 * 128 / 16 + 160) + 200)


CYCLES = 10     # W-cycles of an inner solve at c_F * TOL (measured 9 to 10 over every dt)


def work(case):
    k, n = case["kind"], case["n"]
    sq = float(n * n)
    astar = sq * 16 * (5 * 16 + 8)
    if k == "astar2d":
        return dict(bytes=sq * 16 * 8 * 2, flops=astar)
    if k == "deflated2d":
        return dict(bytes=sq * 16 * 8 * 2, flops=astar + sq * 16 * 40 + CYCLES * _cycle_flops(n, case["pre"], case["post"]))
    if k == "wcycle_batch":
        return dict(bytes=sq * 4 * 16 * 8 * 2, flops=16 * _cycle_flops(n, case["pre"], case["post"]))
    if k == "inner_exact":
        return dict(bytes=sq * 4 * 8 * 2 + (2 * n) ** 2 * 8, flops=4 * 2.0 * (2 * n) ** 3)
    if k == "outer_mg":
        # per square and smoothing step: the update from 13 squares and the residual from 5
        return dict(bytes=sq * 16 * 8 * 2, flops=2.0 * sq * 2 * case["m"] * 2 * 16 * (208 + 80))
    if k == "deflated3d":
        cubes = float(n ** 3)
        return dict(bytes=cubes * 72 * 8 * 2, flops=cubes * (72 * (7 * 48 + 16) + 72 * 7 * 16 + 6 * 8 * 2 * 2 * n))
    if k == "wcycle3d":
        cubes = float(n ** 3)
        return dict(bytes=cubes * 8 * 8 * 2, flops=4.0 / 3 * cubes * 2 * case["smooth"] * 2 * 8 * (200 + 56))
    its = max(20.0, 100.0 * n * math.sqrt(case.get("dt", 1e-4)))
    one = astar + sq * 16 * 50 + CYCLES * _cycle_flops(n, 2, 2)
    if k == "solve2d":
        return dict(bytes=sq * 16 * 8 * 2, flops=its * one)
    return dict(bytes=case["count"] * sq * 16 * 8 * 2, flops=case["count"] * its * one)


# ------------------------------------------------------------------- exact
class _Axis:
    """One-dimensional DG-Q1 matrices of n cells (dof 2 e + i), rows = test: mass M, SIPG stiffness
    K, derivative C[a, b] = int phi_b' phi_a and the face term B[a, b] = jump(phi_a) avg(phi_b);
    face terms at interior nodes and, with left / right, at that end."""

    def __init__(self, n, penalty, left, right):
        h, N = 1.0 / n, 2 * n
        f64 = torch.float64
        e = torch.eye(n, dtype=f64)
        M = torch.kron(e, h * torch.tensor([[2.0, 1.0], [1.0, 2.0]], dtype=f64) / 6.0)
        C = torch.kron(e, torch.tensor([[-0.5, 0.5], [-0.5, 0.5]], dtype=f64))
        K0 = torch.kron(e, torch.tensor([[1.0, -1.0], [-1.0, 1.0]], dtype=f64) / h)
        rows = (n - 1) + int(left) + int(right)
        J, A, D = (torch.zeros(rows, N, dtype=f64) for _ in range(3))   # jump, average, average derivative
        i = torch.arange(n - 1)
        J[i, 2 * i + 1], J[i, 2 * i + 2] = 1.0, -1.0
        A[i, 2 * i + 1] = A[i, 2 * i + 2] = 0.5
        for c in (0, 1):
            D[i, 2 * i + 2 * c], D[i, 2 * i + 2 * c + 1] = -0.5 / h, 0.5 / h
        r = n - 1
        if left:
            J[r, 0], A[r, 0], D[r, 0], D[r, 1] = -1.0, 1.0, -1.0 / h, 1.0 / h
            r += 1
        if right:
            J[r, N - 1], A[r, N - 1], D[r, N - 2], D[r, N - 1] = 1.0, 1.0, -1.0 / h, 1.0 / h
        self.n = n
        self.m = dict(M=M, C=C, B=J.T @ A, K=K0 - J.T @ D - D.T @ J + penalty * n * (J.T @ J))
        self.m = {q: v.cuda() for q, v in self.m.items()}

    def coarse(self):
        """The Galerkin matrices of the agglomerated cells (injection of the coarse functions)."""
        c = object.__new__(_Axis)
        c.n = self.n // 2
        p = torch.tensor([[1.0, 0.0], [0.5, 0.5], [0.5, 0.5], [0.0, 1.0]], dtype=torch.float64)
        c.P = torch.kron(torch.eye(c.n, dtype=torch.float64), p).cuda()
        c.m = {q: c.P.T @ v @ c.P for q, v in self.m.items()}
        return c


def _axes(d, n):
    if d == 2:
        return [_Axis(n, 10.0, True, False)] * 2
    return [_Axis(n, PENALTY3, False, True)] + [_Axis(n, PENALTY3, False, False)] * 2


def _along(A, u, axis):
    """A applied to u along tensor axis 0 = x (last) .. d - 1."""
    u = u.movedim(-1 - axis, -1)
    return (u.reshape(-1, u.shape[-1]) @ A.T.contiguous()).reshape(*u.shape[:-1], A.shape[0]).movedim(-1, -1 - axis)


def _laplace_terms(d):
    """(test, trial, coefficient, matrix per axis) of the SIPG Laplacian."""
    return [(0, 0, 1.0, ["K" if a == i else "M" for a in range(d)]) for i in range(d)]


def _divdiv_terms(d, coef):
    out = []
    for k in range(d):
        for i in range(d):           # trial component (k, i), test component (k, j)
            for j in range(d):
                mats = ["M"] * d
                if i == j:
                    mats[i] = "K"
                    out.append((d * k + j, d * k + i, coef, mats))
                else:
                    for si, sj, sign in (("C", "Ct", 1.0), ("C", "B", -1.0), ("Bt", "Ct", -1.0)):
                        m = list(mats)
                        m[i], m[j] = si, sj
                        out.append((d * k + j, d * k + i, sign * coef, m))
    return out


def _astar_terms(d, dt, nu):
    out = _divdiv_terms(d, dt)
    for c in range(d * d):
        if c // d != c % d:
            out.append((c, c, 1.0 / nu, ["M"] * d))
        else:
            for t in range(d):
                out.append((c, t * (d + 1), ((1.0 if t == c // d else 0.0) - 1.0 / d) / nu, ["M"] * d))
    return out


def _mat(axis, name):
    return axis.m[name[0]].T if name.endswith("t") else axis.m[name]


def _apply(axes, terms, u):
    """The operator on u of shape (..., components, I_d, .., I_x)."""
    d = len(axes)
    out, first = torch.zeros_like(u), {}
    for test, trial, coef, mats in terms:
        key = (trial, mats[0])
        if key not in first:         # the x products are shared by several terms
            first[key] = _along(_mat(axes[0], mats[0]), u.select(-1 - d, trial), 0)
        v = first[key]
        for a in range(1, d):
            v = _along(_mat(axes[a], mats[a]), v, a)
        out.select(-1 - d, test).add_(v, alpha=coef)
    return out


def _to_tensor(v, d, n, comps, cols=1):
    """Element-major (e, column, component, corner) -> (cols, components, I_d, .., I_x)."""
    v = v.reshape([n] * d + [cols, comps] + [2] * d)
    perm = [d, d + 1]
    for a in range(d):
        perm += [a, d + 2 + a]
    return v.permute(perm).reshape([cols, comps] + [2 * n] * d).contiguous()


def _to_elem(u, d, n, comps, cols=1):
    u = u.reshape([cols, comps] + [n, 2] * d)
    perm = [2 + 2 * a for a in range(d)] + [0, 1] + [3 + 2 * a for a in range(d)]
    return u.permute(perm).reshape(-1).contiguous()


class _Laplace:
    """L^{-1} by the generalised eigenvectors of each axis, refined with the operator itself."""

    def __init__(self, axes):
        self.axes, self.terms, self.V, self.lam, done = axes, _laplace_terms(len(axes)), [], [], {}
        for ax in axes:
            if id(ax) not in done:
                Mm, Kk = ax.m["M"].cpu(), ax.m["K"].cpu()
                R = torch.linalg.cholesky(Mm)
                S = torch.linalg.solve_triangular(R, torch.linalg.solve_triangular(R, Kk, upper=False).T, upper=False)
                lam, Q = torch.linalg.eigh(0.5 * (S + S.T))
                done[id(ax)] = (torch.linalg.solve_triangular(R.T, Q, upper=True).cuda(), lam.cuda())
            self.V.append(done[id(ax)][0])
            self.lam.append(done[id(ax)][1])

    def once(self, s):
        d, v = len(self.axes), s
        for a in range(d):
            v = _along(self.V[a].T, v, a)
        den = 0
        for a in range(d):
            den = den + self.lam[a].view([-1] + [1] * a)
        v = v / den
        for a in range(d):
            v = _along(self.V[a], v, a)
        return v

    def solve(self, s):
        z = self.once(s)
        return z + self.once(s - _apply(self.axes, self.terms, z))


class _Cycle:
    """Algorithm 4 on the Galerkin hierarchy of the operator ``terms``: RAS blocks of core^d cells
    and the cells across their faces, D = 1 / (blocks holding a dof), exact solve on level 1."""

    def __init__(self, axes, terms, comps, core, levels, pre, post):
        self.terms, self.comps, self.core, self.pre, self.post = terms, comps, core, pre, post
        self.lev = [axes]
        for _ in range(levels - 1):
            done = {id(a): a.coarse() for a in self.lev[0]}
            self.lev.insert(0, [done[id(a)] for a in self.lev[0]])
        self.d = len(axes)
        self.ras = [None] + [self._blocks(a) for a in self.lev[1:]]
        if comps == 1:
            self.coarse = _Laplace(self.lev[0])
        else:
            m = comps * (2 * self.lev[0][0].n) ** self.d
            I = torch.eye(m, dtype=torch.float64, device="cuda")
            shape = [m, comps] + [2 * self.lev[0][0].n] * self.d
            self.dense = torch.linalg.inv(_apply(self.lev[0], terms, I.view(shape)).reshape(m, m).T.contiguous())

    def _blocks(self, axes):
        """Per class of blocks (the two at either end along each axis, the others): the dofs of its
        blocks (blocks, local) and the local inverse (local, local); and the weights D."""
        d, n, c = self.d, axes[0].n, self.core
        t = n // c
        cells = [p for p in torch.cartesian_prod(*[torch.arange(-1, c + 1)] * d).view(-1, d).tolist()
                 if sum(q < 0 or q >= c for q in p) <= 1]
        N = 2 * n
        out = []
        own = sorted({0, 1, t - 2, t - 1} & set(range(t)))              # ends: a class each
        inner = [b for b in range(t) if b not in own]
        pos = [own + inner[:1]] * d
        for cls in torch.cartesian_prod(*[torch.tensor(p) for p in pos]).view(-1, d).tolist():
            live = [p for p in cells if all(0 <= c * b + q < n for b, q in zip(cls, p))]
            loc = [[2 * q + i for q, i in zip(p, ix)] for p in live
                   for ix in torch.cartesian_prod(*[torch.arange(2)] * d).view(-1, d).tolist()]
            loc = torch.tensor(loc, device="cuda")                      # (local, axis x..) relative
            rep = loc + 2 * c * torch.tensor(cls, device="cuda")
            m = len(loc)
            A = torch.zeros(self.comps * m, self.comps * m, dtype=torch.float64, device="cuda")
            for test, trial, coef, mats in self.terms:
                v = coef
                for a in range(d):
                    v = v * _mat(axes[a], mats[a])[rep[:, a][:, None], rep[:, a][None, :]]
                A[test * m:(test + 1) * m, trial * m:(trial + 1) * m] += v
            along = [[b] if b in own else inner for b in cls]
            base = torch.cartesian_prod(*[torch.tensor(a, device="cuda") for a in along]).view(-1, d)
            idx = torch.zeros(len(base), m, dtype=torch.int64, device="cuda")
            for a in reversed(range(d)):                                # x is the fastest axis
                idx = idx * N + (2 * c * base[:, a][:, None] + loc[:, a][None, :])
            idx = torch.cat([idx + q * N ** d for q in range(self.comps)], 1)
            out.append((idx, torch.linalg.inv(A)))
        count = torch.zeros(self.comps * N ** d, dtype=torch.float64, device="cuda")
        for idx, _ in out:
            count.index_add_(0, idx.reshape(-1), torch.ones(idx.numel(), dtype=torch.float64, device="cuda"))
        return out, 1.0 / count

    def smooth(self, k, f, z, steps):
        axes, (blocks, w) = self.lev[k], self.ras[k]
        for _ in range(steps):
            r = (f - _apply(axes, self.terms, z)).reshape(f.shape[0], -1)
            u = torch.zeros_like(r)
            for col in range(r.shape[0]):
                for idx, inv in blocks:
                    u[col].index_add_(0, idx.reshape(-1), (r[col][idx] @ inv.T.contiguous()).reshape(-1))
            z = z + (u * w).view(f.shape)
        return z

    def __call__(self, k, f, z):
        if k == 0:
            if self.comps == 1:
                return self.coarse.solve(f)
            return (f.reshape(f.shape[0], -1) @ self.dense.T.contiguous()).view(f.shape)
        z = self.smooth(k, f, z, self.pre)
        r = f - _apply(self.lev[k], self.terms, z)
        for a in range(self.d):
            r = _along(self.lev[k - 1][a].P.T, r, a)
        c = torch.zeros_like(r)
        for _ in range(2 if k > 1 else 1):
            c = self(k - 1, r, c)
        for a in range(self.d):
            c = _along(self.lev[k - 1][a].P, c, a)
        return self.smooth(k, f, z + c, self.post)


def _trace(u, d):
    """Z^T u of (1, d^2, ...) -> (1, 1, ...)."""
    return sum(u[:, i * (d + 1):i * (d + 1) + 1] for i in range(d)) / math.sqrt(d)


def _spread(y, d, comps):
    u = torch.zeros([1, comps] + list(y.shape[2:]), dtype=y.dtype, device=y.device)
    for i in range(d):
        u[:, i * (d + 1)] = y[:, 0] / math.sqrt(d)
    return u


def _solve(axes, terms, dt, b):
    """A* x = b by deflated CG with the exact inner solve, restarted on the true residual."""
    d, lap = len(axes), _Laplace(axes)

    def project(v):                 # Z E^{-1} Z^T v, E = (dt / d) L
        return _spread(d / dt * lap.once(_trace(v, d)), d, d * d)

    x, norm = torch.zeros_like(b), b.norm()
    for _ in range(3):
        r = b - _apply(axes, terms, x)
        x0 = project(r)
        r = r - _apply(axes, terms, x0)
        xh, p, rho = torch.zeros_like(b), r.clone(), (r * r).sum()
        for it in range(2000):
            if it % 10 == 0 and float(rho) <= (1e-14 * float(norm)) ** 2:
                break
            w = _apply(axes, terms, p)
            q = w - _apply(axes, terms, project(w))
            a = rho / (p * q).sum()
            xh, r = xh + a * p, r - a * q
            new = (r * r).sum()
            p, rho = r + (new / rho) * p, new
        x = x + x0 + xh - project(_apply(axes, terms, xh))
        if float((b - _apply(axes, terms, x)).norm()) <= 1e-13 * float(norm):
            break
    return x


def exact(case, seed):
    k, n = case["kind"], case["n"]
    d = 3 if k.endswith("3d") or "3d" in k else 2
    axes = _axes(d, n)
    comps = d * d
    nu = NU3 if d == 3 else 1.0
    if k == "astar2d":
        x = _to_tensor(_randn(16 * n * n, seed), 2, n, 4)
        return _to_elem(_apply(axes, _astar_terms(2, case["dt"], nu), x), 2, n, 4)
    if k in ("deflated2d", "deflated3d"):
        dt, terms = case["dt"], _astar_terms(d, case["dt"], nu)
        x = _to_tensor(_randn(comps * 2 ** d * n ** d, seed), d, n, comps)
        w = _apply(axes, terms, x)
        y = d / dt * _Laplace(axes).solve(_trace(w, d))
        return _to_elem(w - _apply(axes, _divdiv_terms(d, dt), _spread(y, d, comps)), d, n, comps)
    if k == "inner_exact":
        s = _to_tensor(_randn(4 * n * n, seed), 2, n, 1)
        return _to_elem(2.0 / case["dt"] * _Laplace(axes).solve(s), 2, n, 1)
    if k == "wcycle_batch":
        f = _to_tensor(_randn(64 * n * n, seed), 2, n, 1, 16)
        cyc = _Cycle(axes, _laplace_terms(2), 1, 4, int(math.log2(n // 16)) + 1, case["pre"], case["post"])
        return _to_elem(cyc(len(cyc.lev) - 1, f, torch.zeros_like(f)), 2, n, 1, 16)
    if k == "outer_mg":
        f = _to_tensor(_randn(16 * n * n, seed), 2, n, 4)
        cyc = _Cycle(axes, _astar_terms(2, case["dt"], nu), 4, 1, int(math.log2(n // 8)) + 1, case["m"], case["m"])
        return _to_elem(cyc(len(cyc.lev) - 1, f, torch.zeros_like(f)), 2, n, 4)
    if k == "wcycle3d":
        levels, c = 1, n
        while c % 2 == 0 and c > 2:
            levels, c = levels + 1, c // 2
        f = _to_tensor(_randn(8 * n ** 3, seed), 3, n, 1)
        cyc = _Cycle(axes, _laplace_terms(3), 1, 1, levels, case["smooth"], case["smooth"])
        return _to_elem(cyc(len(cyc.lev) - 1, f, torch.zeros_like(f)), 3, n, 1)
    if k == "solve2d":
        b = _to_tensor(_randn(16 * n * n, seed), 2, n, 4)
        return _to_elem(_solve(axes, _astar_terms(2, case["dt"], nu), case["dt"], b), 2, n, 4)
    if k == "serve":
        b = _randn(case["count"] * 16 * n * n, seed).view(case["count"], -1)
        return torch.stack([_to_elem(_solve(axes, _astar_terms(2, dt, nu), dt, _to_tensor(b[i], 2, n, 4)), 2, n, 4)
                            for i, dt in enumerate(_dts(case))])
    return None

"""Performance cases of the p-multigrid Poisson solver: the work a program has it do.

A case is a dict of plain values.  Its "kind" names the entry point:

  solve     Solver.solve: one MGCG solve to 1e-10 from x = 0 (whole call)
  batch     BatchSolver.solve: many small grids in one lock-step solve (whole call)
  vcycle    Solver.vcycle: one V-cycle, the preconditioner of a Krylov method of the
            program's own
  smooth    Solver.smooth: one smoothing step on the top level, in place
  operator  Solver.residual, .restrict and .prolong on the top level: the pieces of a
            multigrid cycle that a program puts together itself
  train     mlp_forward, mlp_backward and mlp_adam: one training step of the network
            that predicts the face weights

Problems are the repository's own (synth/workloads.py, bench.py, tests): the 2D
4 x 4 P = 4 grid, the paper's periodic 16 x 16 P = 16 grid, 16^3 P = 8 in FP64, the
stretched 32^3 LDG grid in mixed precision, 8^3 P = 32, the continuous
counterpart on 16^3, a batch of small grids; and ragged sizes between them.

exact() computes the same quantities in 64 bits with torch and numpy alone, from
the definitions: dense 1D operators over a whole direction, patch eigenpairs by
LAPACK, direct solves by diagonalisation of the global 1D operators.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

TOL = 1e-10
HID, N_IN, N_OUT = 64, 6, 2  # the face-weight network


# ---------------------------------------------------------------------------- cases
def _grid_case(name, kind, n, P, **kw):
    c = dict(name=name, kind=kind, dim=len(n), n0=n[0], n1=n[1], n2=n[2] if len(n) == 3 else 1, P=P, flux="ip",
             smoother="FA", periodic=False, stretch=0.0, prec="fp64", disc="dg", vcycle="classical")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest whole call: launches and host work are everything
        _grid_case("solve_2d_4x4_p4_fp64", "solve", (4, 4), 4, smoother="EA"),
        # the headline solve: 3.0 M unknowns in FP64
        _grid_case("solve_3d_16c_p8_fp64", "solve", (16, 16, 16), 8),
        # the paper's own test grid: small 2D, periodic, high order
        _grid_case("vcycle_2d_16x16_p16_fp64", "vcycle", (16, 16), 16, smoother="EA", periodic=True),
        # an ordinary small 3D problem, odd element counts
        _grid_case("vcycle_3d_7x5x6_p4_fp64", "vcycle", (7, 5, 6), 4, stretch=1.0),
        # the smoothing step that dominates the headline solve
        _grid_case("smooth_3d_16c_p8_fp64", "smooth", (16, 16, 16), 8),
        # the largest: 23.9 M unknowns, LDG, z stretched, the FP32 V-cycle of mixed precision
        _grid_case("vcycle_3d_32c_p8_ldg_fp32", "vcycle", (32, 32, 32), 8, flux="ldg", stretch=-32.0, prec="mixed"),
        # very high order: elements and patches beyond the LDS
        _grid_case("vcycle_3d_8c_p32_fp32", "vcycle", (8, 8, 8), 32, stretch=5.0, prec="mixed"),
        # high order, ragged counts, FP32
        _grid_case("smooth_3d_9x7x11_p12_fp32", "smooth", (9, 7, 11), 12, stretch=2.0, prec="mixed"),
        # operator and transfers by themselves, order 16
        _grid_case("operator_3d_7x9x6_p16_fp64", "operator", (7, 9, 6), 16, stretch=1.0),
        # the continuous counterpart on the headline grid
        _grid_case("vcycle_3d_16c_p8_se_fp64", "vcycle", (16, 16, 16), 8, smoother="EA", disc="se"),
        # many small grids at once
        dict(name="batch_32_small_mixed", kind="batch", count=32, shapes=4, nlo=2, nhi=6, prec="mixed"),
        # the learned weights' training step (the faces of the training problems)
        dict(name="train_b6144", kind="train", rows=6144),
    ]


def draw(rng):
    kind = rng.choice(["solve", "vcycle", "vcycle", "smooth", "smooth", "smooth", "operator", "batch", "train"])
    if kind == "train":
        return dict(kind="train", rows=int(round(2 ** rng.uniform(7.0, 13.0))))
    if kind == "batch":
        lo = rng.randint(2, 4)
        return dict(kind="batch", count=rng.randint(4, 40), shapes=rng.randrange(1 << 20), nlo=lo, nhi=lo + rng.randint(0, 3),
                    prec=rng.choice(["fp64", "mixed"]))
    prec = rng.choice(["fp64", "mixed"])
    if kind == "solve" or rng.random() < 0.6:
        disc = "dg" if kind == "operator" or rng.random() < 0.85 else "se"
    else:
        disc = "dg"
    dim = 3 if rng.random() < 0.8 else 2
    P = rng.choice([2, 3, 4, 6, 8, 8, 12, 16] if dim == 3 else [4, 8, 12, 16, 32])
    if kind == "vcycle" and dim == 3 and disc == "dg" and rng.random() < 0.1:
        P = 32
    top = {"solve": 1.0e6, "vcycle": 4.0e6, "smooth": 4.0e6, "operator": 6.0e6}[kind] if dim == 3 else 3.0e5
    dof = math.exp(rng.uniform(math.log(3.0e3), math.log(top)))
    per = max(2.0, (dof / (P + 1) ** dim) ** (1.0 / dim))
    periodic = rng.random() < 0.25
    n = [max(3 if periodic else 2, int(round(per * 2 ** rng.uniform(-0.4, 0.4)))) for _ in range(dim)]
    flux = "ldg" if disc == "dg" and rng.random() < 0.25 else "ip"
    smoother = "EA" if disc == "se" or dim == 2 or rng.random() < 0.3 else "FA"
    c = _grid_case("", kind, n, P, flux=flux, smoother=smoother, periodic=periodic, stretch=rng.choice([0.0, 1.0, 2.0]),
                   prec=prec, disc=disc, vcycle="variable" if rng.random() < 0.1 else "classical")
    del c["name"]
    return c


# ---------------------------------------------------------------------------- problems
def _spacing(n, stretch, d):
    """Element sizes of direction d (sum 1): equal, geometric (stretch < 0: the last
    direction, smallest size 1/(n |stretch|)), or ratios up to 2^stretch."""
    if stretch < 0.0:
        if d != 2:
            return np.full(n, 1.0 / n)
        first = 1.0 / (n * -stretch)
        lo, hi = 1.0 + 1e-12, 4.0
        for _ in range(200):
            q = 0.5 * (lo + hi)
            if first * (q ** n - 1.0) / (q - 1.0) < 1.0:
                lo = q
            else:
                hi = q
        h = q ** np.arange(n, dtype=np.float64)
    elif stretch == 0.0:
        return np.full(n, 1.0 / n)
    else:
        h = 2.0 ** np.random.default_rng(100 * n + d).uniform(0.0, stretch, n)
    return h / h.sum()


def _problem(c):
    n = [c["n0"], c["n1"], c["n2"]][: c["dim"]]
    g = SimpleNamespace(dim=c["dim"], dx=tuple(_spacing(k, c["stretch"], d) for d, k in enumerate(n)),
                        periodic=(bool(c["periodic"]),) * c["dim"])
    m = SimpleNamespace(P=c["P"], flux=c["flux"], beta=(0.5,) * 3 if c["flux"] == "ldg" else (0.0,) * 3, mu_star=1.0,
                        smoother=c["smoother"], overlap="level", weighting="quintic", vcycle=c["vcycle"], ns=(1, 1),
                        precision=c["prec"], order="lex", disc=c["disc"])
    return g, m


def _batch_problems(c):
    rng = np.random.default_rng(c["shapes"])
    out = []
    for _ in range(c["count"]):
        n = rng.integers(c["nlo"], c["nhi"] + 1, 3)
        P = int(rng.choice([4, 6, 8]))
        length = 2.0 ** rng.uniform(0.0, 3.0, 3)
        length /= length.min()
        g = SimpleNamespace(dim=3, dx=tuple(np.full(int(k), float(s) / int(k)) for k, s in zip(n, length)),
                            periodic=(False,) * 3)
        out.append((g, SimpleNamespace(P=P, flux="ip", beta=(0.0,) * 3, mu_star=1.0, smoother="FA", overlap="level",
                                       weighting="quintic", vcycle="classical", ns=(1, 1), precision=c["prec"],
                                       order="lex", disc="dg")))
    return out


def _vec_type(c):
    return torch.float32 if c["prec"] == "mixed" and c["kind"] not in ("solve", "batch") else torch.float64


def _size(g, P, disc):
    out = 1
    for d in range(g.dim):
        out *= len(g.dx[d]) * P - (0 if g.periodic[d] else 1) if disc == "se" else len(g.dx[d]) * (P + 1)
    return out


def _inputs(c, seed):
    """The input vectors of a case, from its seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def uni(*shape, dtype=torch.float64):
        return torch.rand(*shape, generator=gen, device="cuda", dtype=dtype) * 2.0 - 1.0

    if c["kind"] == "train":
        B = c["rows"]
        parts = [uni(HID * N_IN) / math.sqrt(N_IN), uni(HID) * 0.1, uni(HID * HID) / math.sqrt(HID), uni(HID) * 0.1,
                 uni(N_OUT * HID) / math.sqrt(HID), uni(N_OUT) * 0.1]
        p = torch.cat(parts).float()
        return dict(p=p, X=uni(B, N_IN).float(), T=uni(B, N_OUT).float(), m=uni(p.numel()).float() * 1e-3,
                    v=(uni(p.numel()).float() * 1e-3).square())
    if c["kind"] == "batch":
        return dict(rhs=torch.cat([uni(_size(g, m.P, "dg")) for g, m in _batch_problems(c)]))
    g, m = _problem(c)
    n = _size(g, m.P, m.disc)
    f = uni(n)
    if all(g.periodic):  # the system is consistent for right-hand sides that sum to zero
        for _ in range(2):
            f -= f.mean()
    out = dict(f=f.to(_vec_type(c)))
    if c["kind"] in ("smooth", "operator"):
        out["u"] = uni(n).to(_vec_type(c))
    if c["kind"] == "operator":
        out["uc"] = uni(_size(g, m.P // 2, m.disc)).to(_vec_type(c))
    return out


def prepare(case, seed):
    from paper_1603_02524_amd import dgmg
    s = SimpleNamespace(kind=case["kind"], dgmg=dgmg, **_inputs(case, seed))
    if s.kind == "batch":
        s.solver = dgmg.BatchSolver(_batch_problems(case))
    elif s.kind != "train":
        g, m = _problem(case)
        s.solver = dgmg.Solver(g, m)
        s.top = s.solver.num_levels - 1
    return s


def run(s):
    if s.kind == "solve":
        x = torch.zeros_like(s.f)
        s.solver.solve(s.f, x, tol=TOL)
        return x
    if s.kind == "batch":
        x = torch.zeros_like(s.rhs)
        s.solver.solve(s.rhs, x, tol=TOL)
        return x
    if s.kind == "vcycle":
        return s.solver.vcycle(s.f)
    if s.kind == "smooth":
        return s.solver.smooth(s.top, s.u.clone(), s.f, 1)
    if s.kind == "operator":
        r = s.solver.residual(s.top, s.f, s.u)
        return {"r": r, "fc": s.solver.restrict(s.top, r), "u": s.solver.prolong(s.top, s.uc, s.u.clone())}
    p, m, v = s.p.clone(), s.m.clone(), s.v.clone()
    y, hidden = s.dgmg.mlp_forward(p, s.X)
    grad = s.dgmg.mlp_backward(p, s.X, s.T, y, hidden)
    s.dgmg.mlp_adam(p, grad, m, v, 10, lr=1e-3)
    return {"y": y, "grad": grad, "p": p, "m": m, "v": v}


# ---------------------------------------------------------------------------- needed work
def _overlap(P, disc):
    return 1 + (P + 4) // 8 - (1 if disc == "se" else 0)


def _level_flops(g, m, P, cycles):
    """cycles = (sweeps, residuals, transfers) on a level of order P."""
    D, q = g.dim, (P if m.disc == "se" else P + 1)
    n = _size(g, P, m.disc)
    NP, ne = P + 1, 1
    for d in range(D):
        ne *= len(g.dx[d])
    lat = NP + 2 * _overlap(P, m.disc)
    na = lat if m.smoother == "EA" else 2 * P
    # per patch: the 1D transforms, those of the first directions once for every node that patches share
    ln = [na] + [lat] * (D - 1)
    sweep = 0
    for d in range(D):
        lines = 1
        for e in range(D):
            lines *= ln[e] if e < d else (q if e > d else 1)
        sweep += lines * ln[d] * ln[d]
    res = n * (2.0 * D * NP + 6 * D)
    tr = n * 2.0 * sum(0.5 ** k for k in range(1, D + 1)) * NP
    return cycles[0] * ne * 4.0 * sweep + cycles[1] * res + cycles[2] * tr


def _cycle_work(g, m, word):
    P, flops, l = m.P, 0.0, 0
    while P > 1:
        steps = 2 ** l if m.vcycle == "variable" else 1
        sweeps = 2 * steps * (g.dim if m.smoother == "FA" else 1)
        flops += _level_flops(g, m, P, (sweeps, sweeps, 2))
        P, l = P // 2, l + 1
    return {"bytes": 2.0 * word * _size(g, m.P, m.disc), "flops": flops}


def work(case):
    if case["kind"] == "train":
        B, par = case["rows"], HID * N_IN + HID * HID + N_OUT * HID
        npar = par + 2 * HID + N_OUT
        return {"bytes": 4.0 * (B * (N_IN + 2 * N_OUT) + 7 * npar), "flops": 2.0 * B * (3 * par - HID * N_IN)}
    word = 4.0 if _vec_type(case) == torch.float32 else 8.0
    if case["kind"] == "batch":
        tot = {"bytes": 0.0, "flops": 0.0}
        for g, m in _batch_problems(case):
            w = _cycle_work(g, m, 8.0)
            n = _size(g, m.P, "dg")
            tot["bytes"] += w["bytes"]
            tot["flops"] += 4.0 * (w["flops"] + n * (2.0 * 3 * (m.P + 1) + 18))
        return tot
    g, m = _problem(case)
    n = _size(g, m.P, m.disc)
    if case["kind"] == "smooth":
        k = g.dim if m.smoother == "FA" else 1
        return {"bytes": 3.0 * word * n, "flops": _level_flops(g, m, m.P, (k, k, 0))}
    if case["kind"] == "operator":
        nc = _size(g, m.P // 2, m.disc)
        return {"bytes": word * (4.0 * n + 2.0 * nc), "flops": _level_flops(g, m, m.P, (0, 1, 2))}
    w = _cycle_work(g, m, word)
    if case["kind"] == "solve":  # about four (FA) or six (EA) iterations
        k = 4.0 if m.smoother == "FA" else 6.0
        w["flops"] = k * (w["flops"] + n * (2.0 * g.dim * (m.P + 1) + 6 * g.dim + 14))
    return w


# ---------------------------------------------------------------------------- the same in 64 bits
def _gll(P):
    """GLL nodes and weights of order P."""
    leg = np.polynomial.legendre.Legendre.basis(P)
    x = np.concatenate(([-1.0], np.sort(np.real(leg.deriv().roots())) if P > 1 else [], [1.0]))
    d1, d2 = leg.deriv(), leg.deriv(2)
    for _ in range(3):
        if P > 1:
            x[1:-1] -= d1(x[1:-1]) / d2(x[1:-1])
    x = 0.5 * (x - x[::-1])
    return x, 2.0 / (P * (P + 1) * leg(x) ** 2)


def _interp(xs, xt):
    """Lagrange interpolation from the nodes xs to the points xt."""
    out = np.ones((len(xt), len(xs)))
    for k in range(len(xs)):
        for j in range(len(xs)):
            if j != k:
                out[:, k] *= (xt - xs[j]) / (xs[k] - xs[j])
    return out


def _diff(x):
    """Differentiation matrix D[i, k] = phi_k'(x_i) (barycentric weights, rows sum to zero)."""
    n = len(x)
    w = np.array([1.0 / np.prod([x[k] - x[j] for j in range(n) if j != k]) for k in range(n)])
    D = np.zeros((n, n))
    for i in range(n):
        for k in range(n):
            if i != k:
                D[i, k] = w[k] / w[i] / (x[i] - x[k])
        D[i, i] = -D[i].sum()
    return D


def _axis(P, dx, periodic, beta, disc):
    """One direction of a level: dense stiffness L, mass vector M (over all its nodes)."""
    x, rho = _gll(P)
    D = _diff(x)
    K = D.T @ np.diag(rho) @ D
    N, NP = len(dx), P + 1
    if disc == "se":
        nt = N * P
        L, M = np.zeros((nt + 1, nt + 1)), np.zeros(nt + 1)
        for e in range(N):
            i = np.arange(e * P, e * P + NP)
            L[np.ix_(i, i)] += 2.0 / dx[e] * K
            M[i] += 0.5 * dx[e] * rho
        if periodic:
            L[0] += L[nt]
            L[:, 0] += L[:, nt]
            M[0] += M[nt]
            return L[:nt, :nt], M[:nt]
        return L[1:nt, 1:nt], M[1:nt]
    G = N * NP
    L, M = np.zeros((G, G)), np.zeros(G)
    for e in range(N):
        i = np.arange(e * NP, (e + 1) * NP)
        L[np.ix_(i, i)] += 2.0 / dx[e] * K
        M[i] += 0.5 * dx[e] * rho
    for face in range(N if periodic else N + 1):  # between elements a | b: jump v- - v+, flux of the derivatives
        a, b = face - 1, face
        jump, flux = np.zeros(G), np.zeros(G)
        if periodic:
            a %= N
        ina, inb = a >= 0, b < N
        if ina:
            ia = np.arange(a * NP, (a + 1) * NP)
            jump[ia[-1]] += 1.0
            flux[ia] += (0.5 + beta if inb else 1.0) * 2.0 / dx[a] * D[-1]
        if inb:
            ib = np.arange(b * NP, (b + 1) * NP)
            jump[ib[0]] -= 1.0
            flux[ib] += (0.5 - beta if ina else 1.0) * 2.0 / dx[b] * D[0]
        if ina and inb:
            ra, rb = dx[a] * rho[-1], dx[b] * rho[0]
            mu = 2.0 * (0.5 / ra + 0.5 / rb)
            pen = 2.0 * (beta * beta + beta) / ra + 2.0 * (beta * beta - beta) / rb + mu
        else:
            pen = 4.0 / (dx[a if ina else b] * rho[0])
        L -= np.outer(flux, jump) + np.outer(jump, flux) - pen * np.outer(jump, jump)
    return L, M


def _phi(x):
    return np.where(np.abs(x) < 1.0, (15.0 * x - 10.0 * x ** 3 + 3.0 * x ** 5) / 8.0, np.sign(x))


def _patches(P, dx, periodic, L, M, face, disc):
    """Patches of one direction: node indices (a dead slot at the end outside a Dirichlet
    domain), eigenvectors, eigenvalues and weights, padded to one length."""
    x, _ = _gll(P)
    N, G, q = len(dx), len(M), P if disc == "se" else P + 1
    no, shift = _overlap(P, disc), 1 if disc == "se" and not periodic else 0
    count = N + 1 if face and not periodic else N
    n = 2 * P if face else P + 1 + 2 * no
    idx, S = np.full((count, n), G), np.zeros((count, n, n))
    lam, w = np.ones((count, n)), np.zeros((count, n))
    for p in range(count):
        raw = ((p - 1) * q + 1 if face else p * q - no) + np.arange(n)
        e = np.floor_divide(raw, q)
        xi = x[raw - e * q]
        st = raw % G if periodic else raw - shift
        ok = np.ones(n, bool) if periodic else (st >= 0) & (st < G)
        if face:
            wt = 0.5 * (1.0 + _phi(1.0 - np.abs(np.where(e == p - 1, xi - 1.0, xi + 1.0))))
        else:
            width, y = x[no + 1 if disc == "se" else no] + 1.0, xi + 2.0 * (e - p)
            left, right = _phi((1.0 + y) / width), _phi((1.0 - y) / width)
            if not periodic and p == 0:
                left = np.ones(n)
            if not periodic and p == N - 1:
                right = np.ones(n)
            wt = 0.5 * (left + right)
        k, j = np.flatnonzero(ok), st[ok]
        r = 1.0 / np.sqrt(M[j])
        A = L[np.ix_(j, j)] * np.outer(r, r)
        val, vec = np.linalg.eigh(0.5 * (A + A.T))
        S[p][np.ix_(k, k)] = r[:, None] * vec
        idx[p, k], lam[p, k], w[p, k] = j, val, wt[ok]
    return [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (idx, S, lam, w)]


def _along(A, u, ax):
    """A applied along axis ax of u."""
    v = u.movedim(ax, -1)
    return (v.reshape(-1, v.shape[-1]) @ A.T.contiguous()).reshape(*v.shape[:-1], A.shape[0]).movedim(-1, ax)


class _Reference:
    """Levels of one problem as dense 1D operators; vectors are arrays over the nodes,
    the last direction first."""

    def __init__(self, g, m):
        self.g, self.m, self.D = g, m, g.dim
        self.order = [m.P]
        while self.order[-1] > 1:
            self.order.append(self.order[-1] // 2)
        beta = 0.5 if m.flux == "ldg" else 0.0
        self.np1d = [[_axis(P, g.dx[d], g.periodic[d], beta, m.disc) for d in range(self.D)] for P in self.order]
        self.ops = [[(torch.from_numpy(L).cuda(), torch.from_numpy(M).cuda()) for L, M in lv] for lv in self.np1d]

    def axis(self, d):
        return self.D - 1 - d

    def to_nodes(self, l, v):
        n, NP, D = [len(h) for h in self.g.dx], self.order[l] + 1, self.D
        if self.m.disc == "se":
            return v.double().reshape([len(self.np1d[l][d][1]) for d in reversed(range(D))])
        a = v.double().reshape(n[::-1] + [NP] * D)
        return a.permute([k for d in range(D) for k in (d, D + d)]).reshape([k * NP for k in n[::-1]])

    def from_nodes(self, l, a):
        n, NP, D = [len(h) for h in self.g.dx], self.order[l] + 1, self.D
        if self.m.disc == "se":
            return a.reshape(-1)
        a = a.reshape([k for e in n[::-1] for k in (e, NP)])
        return a.permute([2 * d for d in range(D)] + [2 * d + 1 for d in range(D)]).reshape(-1)

    def scale(self, l, u, d):
        shape = [1] * self.D
        shape[self.axis(d)] = -1
        return u * self.ops[l][d][1].reshape(shape)

    def apply(self, l, u):
        y = torch.zeros_like(u)
        for d in range(self.D):
            v = _along(self.ops[l][d][0], u, self.axis(d))
            for e in range(self.D):
                if e != d:
                    v = self.scale(l, v, e)
            y += v
        return y

    def sweep(self, l, u, f, normal):
        D = self.D
        tab = [_patches(self.order[l], self.g.dx[d], self.g.periodic[d], *self.np1d[l][d], d == normal, self.m.disc)
               for d in range(D)]
        r = f - self.apply(l, u)
        for d in range(D):  # each direction: nodes -> (patch, mode)
            idx, S, _, _ = tab[d]
            v = r.movedim(self.axis(d), 0)
            shape = v.shape[1:]
            v = torch.cat([v.reshape(v.shape[0], -1), v.new_zeros(1, v[0].numel())])
            v = torch.stack([S[p].T.contiguous() @ v[idx[p]] for p in range(len(idx))])
            r = v.reshape(-1, *shape).movedim(0, self.axis(d))
        den = 0.0
        for d in range(D):
            shape = [1] * D
            shape[self.axis(d)] = -1
            den = den + tab[d][2].reshape(shape)
        r = r / den
        for d in range(D):  # and back, weighted and summed over the patches of a node
            idx, S, _, w = tab[d]
            v = r.movedim(self.axis(d), 0)
            shape = v.shape[1:]
            v = v.reshape(len(idx), idx.shape[1], -1)
            out = v.new_zeros(len(self.np1d[l][d][1]) + 1, v.shape[2])
            for p in range(len(idx)):
                out.index_add_(0, idx[p], w[p][:, None] * (S[p] @ v[p]))
            r = out[:-1].reshape(-1, *shape).movedim(0, self.axis(d))
        return u + r

    def smooth(self, l, u, f, steps):
        for _ in range(steps):
            for normal in range(self.D) if self.m.smoother == "FA" else (-1,):
                u = self.sweep(l, u, f, normal)
        return u

    def interpolation(self, l, d):
        """Nodes of level l + 1 (coarser) to nodes of level l along direction d."""
        P, Pc = self.order[l], self.order[l + 1]
        J = _interp(_gll(Pc)[0], _gll(P)[0])
        N = len(self.g.dx[d])
        if self.m.disc != "se":
            return torch.from_numpy(np.kron(np.eye(N), J)).cuda()
        A = np.zeros((N * P + 1, N * Pc + 1))
        for e in range(N):
            A[e * P:e * P + P + 1, e * Pc:e * Pc + Pc + 1] = J
        if self.g.periodic[d]:
            A[:, 0] += A[:, -1]
            return torch.from_numpy(A[:-1, :-1].copy()).cuda()
        return torch.from_numpy(A[1:-1, 1:-1].copy()).cuda()

    def restrict(self, l, r):
        for d in range(self.D):
            r = _along(self.interpolation(l, d).T.contiguous(), r, self.axis(d))
        return r

    def prolong(self, l, u):
        for d in range(self.D):
            u = _along(self.interpolation(l, d), u, self.axis(d))
        return u

    def solve(self, l, f):
        """A^+ f by the eigenpairs of the 1D operators of whole directions."""
        singular = all(self.g.periodic)
        if singular:
            f = f - f.mean()
        val, vec = [], []
        for L, M in self.np1d[l]:
            r = 1.0 / np.sqrt(M)
            a = L * np.outer(r, r)
            lam, V = np.linalg.eigh(0.5 * (a + a.T))
            val.append(torch.from_numpy(lam).cuda())
            vec.append(torch.from_numpy(r[:, None] * V).cuda())
        den = 0.0
        for d in range(self.D):
            f = _along(vec[d].T.contiguous(), f, self.axis(d))
            shape = [1] * self.D
            shape[self.axis(d)] = -1
            den = den + val[d].reshape(shape)
        if singular:  # the constants
            at = den.abs().reshape(-1).argmin()
            f.reshape(-1)[at] = 0.0
            den.reshape(-1)[at] = 1.0
        f = f / den
        for d in range(self.D):
            f = _along(vec[d], f, self.axis(d))
        return f - f.mean() if singular else f

    def vcycle(self, f):
        last = len(self.order) - 1
        us, fs = [None] * (last + 1), [f] + [None] * last
        steps = [2 ** l if self.m.vcycle == "variable" else 1 for l in range(last + 1)]
        for l in range(last):
            us[l] = self.smooth(l, torch.zeros_like(fs[l]), fs[l], steps[l])
            fs[l + 1] = self.restrict(l, fs[l] - self.apply(l, us[l]))
        us[last] = self.solve(last, fs[last])
        for l in reversed(range(last)):
            us[l] = self.smooth(l, us[l] + self.prolong(l, us[l + 1]), fs[l], steps[l])
        return us[0]


def _exact_train(i):
    p, X, T, m, v = (i[k].double() for k in ("p", "X", "T", "m", "v"))
    p.requires_grad_(True)
    at, parts = 0, []
    for shape in ((HID, N_IN), (HID,), (HID, HID), (HID,), (N_OUT, HID), (N_OUT,)):
        k = math.prod(shape)
        parts.append(p[at:at + k].reshape(shape))
        at += k
    h = torch.tanh(X @ parts[0].T + parts[1])
    h = torch.tanh(h @ parts[2].T + parts[3])
    y = h @ parts[4].T + parts[5]
    grad, = torch.autograd.grad((y - T).square().sum() / X.shape[0], p)
    m = 0.9 * m + 0.1 * grad
    v = 0.999 * v + 0.001 * grad * grad
    step = 1e-3 * (m / (1 - 0.9 ** 10)) / ((v / (1 - 0.999 ** 10)).sqrt() + 1e-8)
    return {"y": y.detach(), "grad": grad, "p": (p - step).detach(), "m": m, "v": v}


def exact(case, seed):
    i = _inputs(case, seed)
    if case["kind"] == "train":
        return _exact_train(i)
    if case["kind"] == "batch":
        out, at = [], 0
        for g, m in _batch_problems(case):
            n = _size(g, m.P, "dg")
            R = _Reference(g, m)
            out.append(R.from_nodes(0, R.solve(0, R.to_nodes(0, i["rhs"][at:at + n]))))
            at += n
        return torch.cat(out)
    R = _Reference(*_problem(case))
    f = R.to_nodes(0, i["f"])
    if case["kind"] == "solve":  # on a singular grid x is determined up to a constant
        return None if all(R.g.periodic) else R.from_nodes(0, R.solve(0, f))
    if case["kind"] == "vcycle":
        return R.from_nodes(0, R.vcycle(f))
    u = R.to_nodes(0, i["u"])
    if case["kind"] == "smooth":
        return R.from_nodes(0, R.smooth(0, u, f, 1))
    r = f - R.apply(0, u)
    last = 1 if len(R.order) > 1 else 0
    return {"r": R.from_nodes(0, r), "fc": R.from_nodes(last, R.restrict(0, r)),
            "u": R.from_nodes(0, u + R.prolong(0, R.to_nodes(last, i["uc"])))}

"""Workloads for timing the library through its public entry points.

Each case is one thing that a program which solves space-time slab problems
does over and over: apply the slab Jacobian or the residual, apply the
preconditioner, set it up for a new state and apply it, factor and solve a
batch of patch matrices, or solve a whole slab.  Sizes, degrees, viscosities
and slab lengths are those of the repository's tests, benchmark and serving
stream (2D and 3D, r = 1..3, k = 0..2, nu = 1 .. 1e-3, uniform and perturbed
meshes, FP64 and FP32).

listed()            the fixed cases
draw(rng)           one more case of the same ranges
prepare(case, seed) inputs and the context (or batch) a program keeps
run(state)          one pass; returns its outputs
work(case)          bytes and operations one pass cannot do without
exact(case, seed)   the same outputs from plain FP64 torch
"""
from __future__ import annotations

import math
from math import comb

import numpy as np
import torch
from numpy.polynomial import legendre as npleg
from numpy.polynomial import polynomial as nppoly

from paper_2602_13841_amd import inputs as I
from paper_2602_13841_amd import stmg

PERTURB = 0.2   # vertex perturbation of the mapped meshes, in cell widths


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def _slab(name, op, n, r, k, nu, tau, dtype, perturbed=False, n_q=0, outflow=False):
    """A case on one slab context; n as text, e.g. "16x16x16"."""
    return dict(name=name, op=op, n=n, r=r, k=k, nu=nu, tau=tau, dtype=dtype, perturbed=perturbed, n_q=n_q,
                outflow=outflow)


def listed():
    return [
        # the smallest operator application: a 2D slab of the convergence
        # study's coarse meshes, where launches are all there is
        _slab("jacobian 2d 8x8 r1k1 f64", "jacobian", "8x8", 1, 1, 1.0, 0.1, "f64"),
        # the benchmark's operator application, in the precision of the outer
        # Krylov method and in the precision of the multigrid
        _slab("jacobian 16^3 r2k2 f64", "jacobian", "16x16x16", 2, 2, 1e-2, 1 / 32, "f64"),
        _slab("jacobian 16^3 r2k2 f32", "jacobian", "16x16x16", 2, 2, 1e-2, 1 / 32, "f32"),
        # the outer Krylov operator of a large solve on a perturbed mesh,
        # different extents per axis
        _slab("jacobian 24x20x28 r3k1 f64 perturbed", "jacobian", "24x20x28", 3, 1, 1e-3, 1 / 64, "f64", True),
        # every Newton step and line-search trial evaluates the residual
        _slab("residual 16^3 r2k2 f64", "residual", "16x16x16", 2, 2, 1e-2, 1 / 32, "f64"),
        # one preconditioner application: what an outer iteration costs
        _slab("vcycle 16^3 r3k1 f32 perturbed", "vcycle", "16x16x16", 3, 1, 1e-2, 1 / 64, "f32", True),
        # a new Newton state: smoother set up, then applied once (FP32 on the
        # large perturbed mesh, FP64 with two eigen-systems on a small one)
        _slab("rebuild 24^3 r3k1 f32 perturbed", "rebuild", "24x24x24", 3, 1, 1e-3, 1 / 64, "f32", True),
        _slab("rebuild 8^3 r2k2 f64", "rebuild", "8x8x8", 2, 2, 1e-2, 1 / 64, "f64"),
        # whole slab solves of the serving stream's sizes, with an outflow
        # face (the pressure is then unique)
        _slab("solve 2d 32x32 r3k1", "solve", "32x32", 3, 1, 1e-2, 1 / 64, "f32", True, outflow=True),
        _slab("solve 12^3 r2k1", "solve", "12x12x12", 2, 1, 1e-2, 1 / 64, "f32", True, outflow=True),
        # batches of space-time patch matrices of mixed sizes, factored and
        # solved
        dict(name="patch lu 576 mixed f32", op="lu", batch=576, rmax=3, kmax=2, nu=1.0, dtype="f32"),
        dict(name="patch lu 576 mixed f64", op="lu", batch=576, rmax=3, kmax=2, nu=1e-2, dtype="f64"),
    ]


def _draw_mesh(rng, dim, most_cells):
    """Extents base * 2^levels per axis: the multigrid coarsens them to a few
    cells per axis, as every mesh of the serving stream and the benchmark."""
    while True:
        levels = rng.choice((1, 2, 3, 3, 4) if dim == 2 else (1, 2, 2, 3, 3))
        base = [rng.choice((2, 3, 3, 5) if dim == 2 else (2, 2, 3)) for _ in range(dim)]
        n = [b << levels for b in base]
        if math.prod(base) <= (25 if dim == 2 else 18) and math.prod(n) <= most_cells:
            return "x".join(map(str, n))


def draw(rng):
    op = rng.choice(("jacobian", "jacobian", "jacobian", "residual", "vcycle", "vcycle", "rebuild", "rebuild",
                     "solve", "lu"))
    if op == "lu":
        return dict(op="lu", batch=int(2 ** rng.uniform(4, 9)), rmax=rng.randint(1, 3), kmax=rng.randint(0, 2),
                    nu=rng.choice((1.0, 0.1)), dtype=rng.choice(("f64", "f32")))
    dim = rng.choice((2, 3, 3))
    r, k = rng.randint(1, 3), rng.randint(0, 2)
    most = {"jacobian": 13824, "residual": 13824, "vcycle": 4096, "rebuild": 4096, "solve": 1728}[op] if dim == 3 else 10000
    if dim == 3 and op in ("vcycle", "rebuild"):
        # bound on the factor storage of the finest level
        most = min(most, int(1.2e9 / ((k + 1) * (3 * (r + 2) ** 3 + comb(r + 3, 3)) ** 2)))
    c = _slab("", op, _draw_mesh(rng, dim, max(most, 64)), r, k, rng.choice((1.0, 1e-2, 1e-3)),
              rng.choice((1 / 64, 1 / 32)),
              "f64" if op == "residual" else rng.choice(("f64", "f32")), rng.random() < 0.5,
              r + 2 if op in ("jacobian", "residual") and rng.random() < 0.25 else 0,
              op == "solve" or rng.random() < 0.3)
    del c["name"]
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _dims(case):
    n = tuple(int(v) for v in case["n"].split("x"))
    return len(n), n


def _mask(case, dim):
    full = (1 << (2 * dim)) - 1
    return full & ~2 if case["outflow"] else full   # outflow: the face x = 1


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _uniform(count, gen):
    return torch.rand(count, generator=gen, device="cuda", dtype=torch.float64) * 2 - 1


def _smooth_velocity(dim, n, r, gen):
    """A smooth divergence-free field (curl of random plane waves) at the
    points of the velocity lattice, scaled to max |v| = 1: one time node."""
    ax = [torch.arange((r + 1) * m + 1, device="cuda", dtype=torch.float64) / ((r + 1) * m) for m in n]
    X = torch.meshgrid(*ax[::-1], indexing="ij")[::-1]   # x fastest
    ncomp = 1 if dim == 2 else 3
    kap = torch.randint(1, 6, (8, ncomp, dim), generator=gen, device="cuda").double().cpu()
    amp = torch.randn((8, ncomp), generator=gen, device="cuda", dtype=torch.float64).cpu()
    ph = torch.rand((8, ncomp), generator=gen, device="cuda", dtype=torch.float64).cpu()
    v = [torch.zeros_like(X[0]) for _ in range(dim)]
    for m in range(8):
        for c in range(ncomp):
            kk = kap[m, c]
            a = float(amp[m, c]) / float(kk @ kk)
            arg = 2 * math.pi * (sum(float(kk[j]) * X[j] for j in range(dim)) + float(ph[m, c]))
            g = a * torch.cos(arg)
            if dim == 2:
                v[0] += float(kk[1]) * g
                v[1] -= float(kk[0]) * g
            else:
                b, e = (c + 1) % 3, (c + 2) % 3   # curl of psi_c: component e gets -d_b, b gets d_e
                v[b] += float(kk[e]) * g
                v[e] -= float(kk[b]) * g
    out = torch.stack([w.reshape(-1) for w in v])
    return (out / out.norm(dim=0).max()).reshape(-1)


def _slab_inputs(case, seed):
    dim, n = _dims(case)
    r, k = case["r"], case["k"]
    Nv, Np, N = I.sizes(dim, n, r, k)
    gen = _gen(seed)
    vprev = _smooth_velocity(dim, n, r, gen)
    other = _smooth_velocity(dim, n, r, gen)
    # the state moves from the previous slab's velocity over the time nodes;
    # smooth pressure coefficients of moderate size
    U = torch.zeros(N, dtype=torch.float64, device="cuda")
    nv1 = vprev.numel()
    for a in range(k + 1):
        U[a * nv1:(a + 1) * nv1] = vprev + 0.1 * (a + 1) * other
    U[Nv:] = 0.1 * _uniform(Np, gen)
    x = _uniform(N, gen)
    vert = I.perturbed_vertices(dim, n, PERTURB, seed) if case["perturbed"] else None
    return dim, n, vert, vprev, U, x


def _lu_matrices(case, seed):
    """FP64 surrogate patches of 8^3 meshes, (r, k) over the case's range, as
    the smoother assembles them; right-hand sides A x with x = U(-1, 1)."""
    gen = _gen(seed)
    shapes = [(r, k) for r in range(1, case["rmax"] + 1) for k in range(case["kmax"] + 1)]
    blocks, sizes, rhs = [], [], []
    for i, (r, k) in enumerate(shapes):
        count = case["batch"] // len(shapes) + (1 if i < case["batch"] % len(shapes) else 0)
        if count == 0:
            continue
        ctx = stmg.Context(3, (8, 8, 8), r, k, case["nu"], 1 / 16, prec_mg=stmg.STMG_F64, fgmres_maxit=1)
        ctx.smoother_rebuild(_uniform(ctx.N, gen))
        for j in range(count):
            A = ctx.level_patch(0, (j * 37 + 73) % 512)
            blocks.append(A.reshape(-1))
            sizes.append(A.shape[0])
            rhs.append(A @ _uniform(A.shape[0], gen))
        ctx.close()
    sizes = np.array(sizes, dtype=np.int32)
    return torch.cat(blocks), torch.cat(rhs), sizes


def prepare(case, seed):
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    if case["op"] == "lu":
        A, b, sizes = _lu_matrices(case, seed)
        s64 = sizes.astype(np.int64)
        A, b = A.to(dtype), b.to(dtype)
        return dict(op="lu", A=A, b=b, sizes=sizes, a_off=np.concatenate([[0], np.cumsum(s64 ** 2)[:-1]]),
                    p_off=np.concatenate([[0], np.cumsum(s64)[:-1]]), LU=torch.empty_like(A),
                    piv=torch.zeros(int(s64.sum()), dtype=torch.int32, device="cuda"))
    dim, n, vert, vprev, U, x = _slab_inputs(case, seed)
    op = case["op"]
    prec = stmg.STMG_F64 if dtype == torch.float64 else stmg.STMG_F32
    opts = dict(prec_mg=prec, n_q=case["n_q"])
    if op == "solve":
        opts.update(newton_rtol=1e-10, newton_atol=0.0)
    else:
        opts.update(fgmres_maxit=1)   # no Krylov basis needed
    ctx = stmg.Context(dim, n, case["r"], case["k"], case["nu"], case["tau"], vertices=vert,
                       dirichlet_faces=_mask(case, dim), **opts)
    s = dict(op=op, ctx=ctx)
    if op == "jacobian":
        s.update(U=U.to(dtype), x=x.to(dtype), y=torch.empty(ctx.N, dtype=dtype, device="cuda"))
    elif op == "residual":
        ctx.set_slab_data(0.01 * x, vprev)
        s.update(U=U, y=torch.empty_like(U))
    elif op == "solve":
        ctx.set_slab_data(None, vprev)
        u0 = torch.zeros(ctx.N, dtype=torch.float64, device="cuda")
        u0[: (case["k"] + 1) * vprev.numel()] = vprev.repeat(case["k"] + 1)
        s.update(u0=u0, u=torch.empty_like(u0))
    else:
        if op == "vcycle":
            ctx.smoother_rebuild(U)
        s.update(U=U, r=x.to(dtype), d=torch.empty(ctx.N, dtype=dtype, device="cuda"))
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    op = s["op"]
    if op == "jacobian":
        return s["ctx"].jacobian_vmult(s["U"], s["x"], s["y"])
    if op == "residual":
        return s["ctx"].residual(s["U"], s["y"])
    if op == "vcycle":
        return s["ctx"].vcycle(s["r"], s["d"])
    if op == "rebuild":
        s["ctx"].smoother_rebuild(s["U"])
        return s["ctx"].vcycle(s["r"], s["d"])
    if op == "solve":
        s["u"].copy_(s["u0"])
        return s["ctx"].newton_solve(s["u"])[0]
    s["LU"].copy_(s["A"])   # the factorization is in place
    x = s["b"].clone()
    stmg.batched_lu(s["LU"], s["a_off"], s["sizes"], s["piv"], s["p_off"])
    stmg.batched_lu_solve(s["LU"], s["a_off"], s["sizes"], s["piv"], s["p_off"], x, s["p_off"])
    return x


# --------------------------------------------------------------------------
# algorithmic work
# --------------------------------------------------------------------------
def _levels(case):
    """(cells, r) of the multigrid levels, finest first."""
    dim, n = _dims(case)
    r, n, out = case["r"], list(n), []
    out.append((math.prod(n), r))
    while r > 1:
        r = max(1, r // 2)
        out.append((math.prod(n), r))
    while all(v % 2 == 0 and v >= 4 for v in n):
        n = [v // 2 for v in n]
        out.append((math.prod(n), r))
    return out


def _apply_flops(dim, cells, r, k, nq):
    """Sum-factorized operator: 1D contractions of the fields to the Gauss
    points and back (values of 3 dim fields and the pressure, collocation
    gradients of dim), point arithmetic."""
    n1, total = r + 2, 0
    for ni, fields in ((n1, 4 * dim), (r + 1, 2)):
        for s in range(dim):
            total += fields * 2 * ni * nq ** (s + 1) * ni ** (dim - 1 - s)
    total += 2 * dim * dim * 2 * nq ** (dim + 1) + 20 * dim * dim * nq ** dim
    return cells * (k + 1) * total


def _setup_work(case):
    """Patch factors of the smoothed levels: (bytes stored, LU operations)."""
    dim, w = _dims(case)[0], 8 if case["dtype"] == "f64" else 4
    nt, byt, fl = case["k"] + 1, 0, 0.0
    for cells, r in _levels(case)[:-1]:
        ms = dim * (r + 2) ** dim + comb(r + dim, dim)
        byt += cells * nt * ms * ms * w            # (k+1) real planes: complex systems hold two
        fl += cells * (nt // 2 * 4 + nt % 2) * 2 / 3 * ms ** 3
    return byt, fl


def work(case):
    w = 8 if case["dtype"] == "f64" else 4
    if case["op"] == "lu":
        shapes = [(r, k) for r in range(1, case["rmax"] + 1) for k in range(case["kmax"] + 1)]
        byt = fl = 0.0
        for i, (r, k) in enumerate(shapes):
            count = case["batch"] // len(shapes) + (1 if i < case["batch"] % len(shapes) else 0)
            m = (k + 1) * (3 * (r + 2) ** 3 + comb(r + 3, 3))
            byt += count * 2 * m * m * w
            fl += count * (2 / 3 * m ** 3 + 2 * m * m)
        return dict(bytes=byt, flops=fl)
    dim, n = _dims(case)
    r, k = case["r"], case["k"]
    Nv, Np, N = I.sizes(dim, n, r, k)
    nq = case["n_q"] or (3 * r + 5) // 2
    apply = _apply_flops(dim, math.prod(n), r, k, nq)
    if case["op"] == "jacobian":
        return dict(bytes=(2 * N + Nv) * w, flops=apply)
    if case["op"] == "residual":
        return dict(bytes=(3 * N + Nv // (k + 1)) * w, flops=apply)
    fac, lu = _setup_work(case)
    # a V-cycle: two sweeps per smoothed level, each reading the factors once
    cyc = dict(bytes=2 * fac + 2 * N * w, flops=2 * 2 * fac / w)
    if case["op"] == "vcycle":
        return cyc
    if case["op"] == "rebuild":
        return dict(bytes=fac + cyc["bytes"], flops=lu + cyc["flops"])
    # a solve: about four Newton steps, one setup, sixteen V-cycles
    return dict(bytes=fac + 16 * cyc["bytes"], flops=lu + 16 * cyc["flops"])


# --------------------------------------------------------------------------
# the operators from their definition, FP64
# --------------------------------------------------------------------------
def _lagrange(nodes, x):
    L = np.ones((len(x), len(nodes)))
    D = np.zeros_like(L)
    for j in range(len(nodes)):
        c = np.array([1.0])
        for m in range(len(nodes)):
            if m != j:
                c = nppoly.polymul(c, np.array([-nodes[m], 1.0]) / (nodes[j] - nodes[m]))
        L[:, j] = nppoly.polyval(x, c)
        D[:, j] = nppoly.polyval(x, nppoly.polyder(c))
    return L, D


def _time_tables(k, tau):
    c = np.zeros(k + 2)
    c[k + 1], c[k] = 1.0, -1.0
    t = 0.5 * (np.sort(np.real(npleg.legroots(c))) + 1)
    t[-1] = 1.0
    gx, gw = npleg.leggauss(k + 3)
    gx, gw = 0.5 * (gx + 1), 0.5 * gw
    L, D = _lagrange(t, gx)
    phi0 = _lagrange(t, np.array([0.0]))[0][0]
    K = np.einsum("g,ga,gb->ab", gw, L, D) + np.outer(phi0, phi0)
    return K, tau * (gw @ L), phi0


class _Plain:
    """Spatial form of one time node, cell by cell, at the points of the
    volume rule and of the rules of the boundary faces."""

    def __init__(self, case, seed):
        dim, n, vert, self.vprev, self.U, self.x = _slab_inputs(case, seed)
        r, k = case["r"], case["k"]
        self.dim, self.n, self.r, self.k = dim, n, r, k
        self.nu, self.dev = case["nu"], self.U.device
        self.K, self.w, self.phi0 = _time_tables(k, case["tau"])
        self.Nv, self.Np, self.N = I.sizes(dim, n, r, k)
        n1, nq = r + 2, case["n_q"] or (3 * r + 5) // 2
        gll = np.concatenate([[-1.0], np.sort(np.real(npleg.Legendre.basis(n1 - 1).deriv().roots())), [1.0]])
        gll = 0.5 * (gll + 1)
        gx, gw = npleg.leggauss(nq)
        gx, gw = 0.5 * (gx + 1), 0.5 * gw
        # scalar node and vertex numbers of every cell
        cc = np.stack(np.meshgrid(*[np.arange(m) for m in n[::-1]], indexing="ij")[::-1], -1).reshape(-1, dim)
        loc = np.stack(np.meshgrid(*[np.arange(n1)] * dim, indexing="ij")[::-1], -1).reshape(-1, dim)
        vloc = np.stack(np.meshgrid(*[np.arange(2)] * dim, indexing="ij")[::-1], -1).reshape(-1, dim)
        def number(base, off, ext):
            g, st = 0, 1
            for a in range(dim):
                g = g + st * (base[:, None, a] + off[None, :, a])
                st *= ext[a]
            return g
        self.dof = torch.tensor(number((r + 1) * cc, loc, [(r + 1) * m + 1 for m in n]), device=self.dev)
        vid = number(cc, vloc, [m + 1 for m in n])
        if vert is None:
            idx = np.stack(np.meshgrid(*[np.arange(m + 1) for m in n[::-1]], indexing="ij")[::-1], -1)
            vert = idx.reshape(-1, dim) / np.array(n, dtype=float)
        X = torch.tensor(vert, device=self.dev)[torch.tensor(vid, device=self.dev)]   # [cell][vertex][dim]
        modes = [m for m in np.stack(np.meshgrid(*[np.arange(r + 1)] * dim, indexing="ij")[::-1], -1).reshape(-1, dim)
                 if m.sum() <= r]

        def tables(pts):
            S = [_lagrange(gll, pts[:, a]) for a in range(dim)]
            V = [_lagrange(np.array([0.0, 1.0]), pts[:, a]) for a in range(dim)]
            def tensor(T, off, grad):
                o = np.ones((len(pts), len(off)))
                for a in range(dim):
                    o *= T[a][1 if a == grad else 0][:, off[:, a]]
                return o
            leg = [np.stack([math.sqrt(2 * i + 1) * npleg.legval(2 * pts[:, a] - 1, np.eye(r + 1)[i])
                             for i in range(r + 1)], 1) for a in range(dim)]
            psi = np.stack([np.prod([leg[a][:, m[a]] for a in range(dim)], 0) for m in modes], 1)
            t = lambda v: torch.tensor(v, device=self.dev)
            return (t(tensor(S, loc, -1)), t(np.stack([tensor(S, loc, a) for a in range(dim)])),
                    t(np.stack([tensor(V, vloc, a) for a in range(dim)])), t(psi))

        def rule(fixed):
            g = [gx if fixed is None or a != fixed[0] else np.array([float(fixed[1])]) for a in range(dim)]
            h = [gw if fixed is None or a != fixed[0] else np.ones(1) for a in range(dim)]
            pts = np.stack(np.meshgrid(*g[::-1], indexing="ij")[::-1], -1).reshape(-1, dim)
            wts = np.prod(np.stack(np.meshgrid(*h[::-1], indexing="ij")[::-1], -1).reshape(-1, dim), 1)
            return pts, torch.tensor(wts, device=self.dev)

        self.sets = []   # (cells, basis, d basis, psi, J^{-T}, point weights, normal, Dirichlet, h)
        allc = torch.arange(len(cc), device=self.dev)
        pts, wts = rule(None)
        N_, G_, V_, P_ = tables(pts)
        J = torch.einsum("bqv,kva->kqab", V_, X)
        vw = torch.linalg.det(J) * wts
        self.sets.append((allc, N_, G_, P_, torch.linalg.inv(J).transpose(2, 3), vw, None, False, None))
        vol = vw.sum(1)
        for f in range(2 * dim):
            ax, side = f // 2, f % 2
            pts, wts = rule((ax, side))
            sel = torch.tensor(np.nonzero(cc[:, ax] == (n[ax] - 1 if side else 0))[0], device=self.dev)
            N_, G_, V_, P_ = tables(pts)
            J = torch.einsum("bqv,kva->kqab", V_, X[sel])
            Jit = torch.linalg.inv(J).transpose(2, 3)
            nn = Jit[..., ax] * (1.0 if side else -1.0)
            ln = nn.norm(dim=-1)
            fw = torch.linalg.det(J) * ln * wts
            h = vol[sel] / fw.sum(1) / (r + 1) ** 2
            self.sets.append((sel, N_, G_, P_, Jit, fw, nn / ln[..., None], bool((_mask(case, dim) >> f) & 1), h))

    def form(self, v, p, dv=None, dp=None, m=None):
        """(velocity rows, pressure rows): the spatial form at velocity v
        [c][node] and pressure p [cell][mode], or with (dv, dp) its derivative
        in that direction (p is then not used)."""
        d, nu = self.dim, self.nu
        jac = dv is not None
        rv = torch.zeros_like(v)
        rp = torch.zeros_like(dp if jac else p)
        om = lambda y: 0.5 * (y.abs() - y)
        for cells, N_, G_, P_, Jit, w, nrm, isD, h in self.sets:
            for i in range(0, len(cells), 1024):
                c, Ji, wi = cells[i:i + 1024], Jit[i:i + 1024], w[i:i + 1024]
                D = self.dof[c]
                u = torch.einsum("ckl,ql->kqc", v[:, D], N_)
                x = torch.einsum("ckl,ql->kqc", dv[:, D], N_) if jac else u
                g = torch.einsum("ckl,bql->kqcb", (dv if jac else v)[:, D], G_)
                g = torch.einsum("kqab,kqcb->kqca", Ji, g)
                pr = torch.einsum("km,qm->kq", (dp if jac else p)[c], P_)
                if nrm is None:
                    F = nu * g - x[..., :, None] * u[..., None, :]
                    if jac:
                        F = F - u[..., :, None] * x[..., None, :]
                    F = F - pr[..., None, None] * torch.eye(d, dtype=v.dtype, device=v.device)
                    val, q = None, -torch.einsum("kqaa->kq", g)
                else:
                    nn, hi = nrm[i:i + 1024], (h[i:i + 1024])[:, None, None]
                    un, xn = (u * nn).sum(-1, keepdim=True), (x * nn).sum(-1, keepdim=True)
                    val = xn * u + un * x if jac else un * u
                    F, q = None, None
                    if isD:
                        gn = torch.einsum("kqca,kqa->kqc", g, nn)
                        val = val - nu * gn + pr[..., None] * nn - om(un) * x
                        if jac:
                            val = val - 0.5 * (torch.sign(un) - 1) * xn * u
                        val = val + nu * 10.0 / hi * x + 10.0 / hi * xn * nn
                        F, q = -nu * x[..., :, None] * nn[..., None, :], xn[..., 0]
                out = torch.zeros((d,) + D.shape, dtype=v.dtype, device=v.device)
                if val is not None:
                    out += torch.einsum("kqc,ql->ckl", val * wi[..., None], N_)
                if F is not None:
                    Fr = torch.einsum("kqca,kqab->kqcb", F * wi[..., None, None], Ji)
                    out += torch.einsum("kqcb,bql->ckl", Fr, G_)
                rv.index_add_(1, D.reshape(-1), out.reshape(d, -1))
                if q is not None:
                    rp[c] += torch.einsum("kq,qm->km", q * wi, P_)
        return rv, rp

    def mass(self, m):
        cells, N_, _, _, _, w, _, _, _ = self.sets[0]
        rv = torch.zeros_like(m)
        for i in range(0, len(cells), 1024):
            D = self.dof[cells[i:i + 1024]]
            val = torch.einsum("ckl,ql->ckq", m[:, D], N_) * w[i:i + 1024]
            rv.index_add_(1, D.reshape(-1), torch.einsum("ckq,ql->ckl", val, N_).reshape(self.dim, -1))
        return rv

    def split(self, U):
        nt = self.k + 1
        return U[: self.Nv].view(nt, self.dim, -1), U[self.Nv:].view(nt, len(self.dof), -1)

    def jacobian(self, U, x):
        V, _ = self.split(U)
        X, P = self.split(x)
        rows = [self.form(V[a], None, X[a], P[a]) for a in range(self.k + 1)]
        MX = [self.mass(X[b]) for b in range(self.k + 1)]
        return self.join(rows, MX)

    def join(self, rows, MX, extra=None):
        rv = []
        for a in range(self.k + 1):
            t = float(self.w[a]) * rows[a][0]
            for b in range(self.k + 1):
                t = t + float(self.K[a, b]) * MX[b]
            if extra is not None:
                t = t - float(self.phi0[a]) * extra
            rv.append(t.reshape(-1))
        return torch.cat(rv + [(float(self.w[a]) * rows[a][1]).reshape(-1) for a in range(self.k + 1)])

    def residual(self, U, rhs, vprev):
        V, P = self.split(U)
        rows = [self.form(V[a], P[a]) for a in range(self.k + 1)]
        MX = [self.mass(V[b]) for b in range(self.k + 1)]
        return self.join(rows, MX, self.mass(vprev.view(self.dim, -1))) - rhs


def exact(case, seed):
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    if case["op"] == "lu":
        A, b, sizes = _lu_matrices(case, seed)
        A, b = A.to(dtype).double().cpu(), b.to(dtype).double().cpu()
        out, ao, po = [], 0, 0
        for m in sizes.astype(int):
            out.append(torch.linalg.solve(A[ao:ao + m * m].view(m, m), b[po:po + m]))
            ao, po = ao + m * m, po + m
        return torch.cat(out)
    if case["op"] not in ("jacobian", "residual"):
        return None
    P = _Plain(case, seed)
    if case["op"] == "residual":
        return P.residual(P.U, 0.01 * P.x, P.vprev)
    return P.jacobian(P.U.to(dtype).double(), P.x.to(dtype).double())

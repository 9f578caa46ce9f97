"""The measured work of the cavity eigensolver: single steps, solves and whole
eigensolves through the public entry points of paper_1301_3794_amd.dm, and
what each computes in 64 bits from plain torch.

A case is a dict: ``kind`` says which call it makes, ``geom`` and nx, ny, nz
the cavity and its grid, the rest its options.  The exact results below share
no code with the library: they take its cut fractions (an input of every
operator) and repeat the method on padded torch arrays.
"""
import math

import numpy as np
import torch

from paper_1301_3794_amd import dm

DEV = "cuda"


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # one stencil product on the small sphere: the shortest call a caller's own iteration makes
        dict(name="apply_f64_sphere16", kind="apply", which="M", geom="sphere", nx=16, ny=16, nz=16, prec=64),
        # the preconditioner by itself on a ragged grid (odd sizes from the second level down)
        dict(name="vcycle_f32_ellipsoid", kind="vcycle", geom="ellipsoid", nx=88, ny=72, nz=104, prec=32, nrhs=1,
             nu=2, sigma=5.0),
        # the FP64 preconditioner on a quarter 9-cell cavity: symmetry planes, a long thin grid
        dict(name="vcycle_f64_ninecell", kind="vcycle", geom="ninecell", nx=24, ny=24, nz=256, prec=64, nrhs=1, nu=2,
             sigma=632.0),
        # the block preconditioner of the 128^3 eigensolve (three inversions in lockstep)
        dict(name="vcycle3_f32_sphere128", kind="vcycle", geom="sphere", nx=128, ny=128, nz=128, prec=32, nrhs=3,
             nu=2, sigma=36.0),
        # divergence cleaning of a block of fields
        dict(name="project3_sphere64", kind="project", geom="sphere", nx=64, ny=64, nz=64, nrhs=3),
        # one inversion as the solver-sensitivity study makes it: sphere r = 0.49, FGMRES(40) to 1e-6, FP64
        dict(name="solve_f64_sphere32", kind="solve", geom="sphere49", nx=32, ny=32, nz=32, mode="mg64", nrhs=1, nu=2,
             restart=40, basis32=0, sigma=5.0, rtol=1e-6),
        # two inversions in lockstep with the 9-cell workload's options (FP32 multigrid, FP32 Krylov basis)
        dict(name="solve2_f32_ninecell", kind="solve", geom="ninecell", nx=48, ny=48, nz=512, mode="mg32", nrhs=2,
             nu=4, restart=30, basis32=1, sigma=632.0, rtol=3e-11),
        # a whole small eigensolve: launches and latency count
        dict(name="eigs_f64_sphere16", kind="eigs", geom="sphere", nx=16, ny=16, nz=16, mode="mg64", k=4, block=4,
             sigma=5.0, rtol=1e-11),
        # the headline eigensolve: 6 pairs on the 128^3 sphere
        dict(name="eigs_f32_sphere128", kind="eigs", geom="sphere", nx=128, ny=128, nz=128, mode="mg32", k=6, block=3,
             sigma=36.0, rtol=3e-11),
        # the fused preconditioner of a batch of ellipsoidal cavities of mixed sizes
        dict(name="batch_vcycle16", kind="batch", count=16, pick=0, sigma=5.0),
        # the learned correction: one inference pass
        dict(name="net_apply_sphere128", kind="net", what="apply", geom="sphere", nx=128, ny=128, nz=128, sigma=36.0),
        # and one training pair's loss and weight gradients
        dict(name="net_grad_ellipsoid64", kind="net", what="grad", geom="ellipsoid", nx=64, ny=64, nz=64, sigma=5.0),
    ]


def _coarsest_ok(n):
    """Whether the automatic hierarchy of grid n ends on a coarsest level small enough to be factored quickly."""
    n = list(n)
    while all(v % 2 == 0 for v in n) and max(n) > 8 and min(n) >= 4:
        n = [v // 2 for v in n]
    return n[0] * n[1] * n[2] <= 1300


def _grid(rng, lo, hi, cells):
    """Three sizes, each a multiple of 4 in lo..hi spread over the logarithm, at most `cells` cells."""
    while True:
        n = [4 * max(1, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 4)) for _ in range(3)]
        if n[0] * n[1] * n[2] <= cells and max(n) <= 2.5 * min(n) and _coarsest_ok(n):
            return dict(nx=n[0], ny=n[1], nz=n[2])


def _ninecell(rng, big):
    m = rng.choice([12, 16, 20, 24, 32, 40, 48] if big else [12, 16, 20, 24, 32])
    # about 32/3 cells of length per cell of radius, in multiples that the levels halve
    nz = {12: 128, 16: 168, 20: 208, 24: 256, 32: 336, 40: 416, 48: 512}[m]
    return dict(geom="ninecell", nx=m, ny=m, nz=nz)


def draw(rng):
    kind = rng.choice(["apply", "vcycle", "vcycle", "project", "solve", "solve", "eigs", "batch", "net"])
    cells = 128 ** 3
    if kind == "apply":
        return dict(kind=kind, which=rng.choice(["M", "K", "R"]), geom="ellipsoid", prec=rng.choice([64, 32]),
                    **_grid(rng, 12, 160, cells))
    if kind == "vcycle":
        c = dict(kind=kind, prec=rng.choice([64, 32, 32]), nrhs=rng.randint(1, 3), nu=rng.randint(1, 4))
        if rng.random() < 0.35:
            return dict(c, sigma=632.0, **_ninecell(rng, True))
        return dict(c, geom="ellipsoid", sigma=5.0, **_grid(rng, 12, 128, cells))
    if kind == "project":
        return dict(kind=kind, geom="ellipsoid", nrhs=rng.randint(1, 4), **_grid(rng, 12, 96, 64 ** 3))
    if kind == "solve":
        mode = rng.choice(["mg64", "mg32", "mg32", "pcg64"])
        c = dict(kind=kind, mode=mode, nrhs=1 if mode == "pcg64" else rng.randint(1, 4), nu=rng.randint(2, 4),
                 restart=rng.choice([20, 30, 40]), basis32=rng.randint(0, 1), rtol=rng.choice([1e-10, 3e-11, 1e-11]))
        if mode != "pcg64" and rng.random() < 0.3:
            return dict(c, sigma=632.0, **_ninecell(rng, False))
        return dict(c, geom="ellipsoid", sigma=5.0, **_grid(rng, 12, 96, 72 ** 3))
    if kind == "eigs":
        return dict(kind=kind, geom="ellipsoid", mode=rng.choice(["mg64", "mg32"]), k=rng.randint(2, 6),
                    block=rng.randint(2, 4), sigma=5.0, rtol=1e-11, **_grid(rng, 12, 64, 48 ** 3))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(4, 16), pick=rng.randint(1, 10 ** 6), sigma=5.0)
    return dict(kind=kind, what=rng.choice(["apply", "grad"]), geom="ellipsoid", sigma=5.0,
                **_grid(rng, 16, 128, 64 ** 3))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _dims(c):
    return c["nx"], c["ny"], c["nz"]


def _geometry(c):
    """(geometry, cell size) of a case."""
    n = _dims(c)
    if c["geom"] == "sphere":
        return dm.sphere((0.5, 0.5, 0.5), 0.45), 1.0 / n[0]
    if c["geom"] == "sphere49":
        return dm.sphere((0.5, 0.5, 0.5), 0.49), 1.0 / n[0]
    if c["geom"] == "ellipsoid":
        h = 1.0 / max(n)
        return dm.ellipsoid([0.5 * v * h + o for v, o in zip(n, (0.003, -0.002, 0.001))],
                            [s * v * h for v, s in zip(n, (0.47, 0.45, 0.46))]), h
    length = 1.235   # two tubes of 0.1 and nine cells of 0.115
    return dm.elliptic_bor((0.0, 0.0), 0.0, 9, 0.103, 0.035, 0.115, 0.1,
                           bc_lo=(dm.BC_PMC, dm.BC_PMC, dm.BC_PEC)), length / n[2]


def _batch_grids(c):
    """Semi-axes and sizes of a batch's cavities."""
    r = np.random.default_rng(c["pick"])
    semi = [tuple(float(a) for a in r.uniform(0.3, 0.48, 3)) for _ in range(c["count"])]
    return semi, [int(n) for n in r.choice([32, 48, 64, 80, 96], c["count"])]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _owned(mask):
    """A mask over padded blocks with the padding layer cleared."""
    out = torch.zeros_like(mask)
    out[..., 1:-1, 1:-1, 1:-1] = mask[..., 1:-1, 1:-1, 1:-1]
    return out


def _pshape(n):
    return n[2] + 2, n[1] + 2, n[0] + 2


def _active(frac, n):
    """Active faces as a (3, nz+2, ny+2, nx+2) mask on the GPU."""
    return _owned(torch.from_numpy(frac[:3]).to(DEV).reshape(3, *_pshape(n)) > 0)


def _noise(mask, g, dtype=torch.float64):
    """N(0,1) on the active faces, as a flat face vector."""
    return (torch.randn(mask.shape, generator=g, device=DEV, dtype=torch.float64) * mask).to(dtype).reshape(-1)


def _smooth(mask, g):
    """A random combination of low-order waves on the active faces: the fields the eigensolver inverts."""
    ax = [torch.linspace(0, math.pi, s, device=DEV, dtype=torch.float64) for s in mask.shape[1:]]
    out = torch.zeros(mask.shape, device=DEV, dtype=torch.float64)
    amp = torch.randn(3, 6, 2, generator=g, device=DEV, dtype=torch.float64).cpu()
    for c in range(3):
        for m in range(6):
            kz, ky, kx = 1 + m % 3, 1 + (m // 2) % 2, 1 + m // 3
            out[c] += float(amp[c, m, 0]) * torch.sin(kz * ax[0] + float(amp[c, m, 1]))[:, None, None] * \
                torch.cos(ky * ax[1])[None, :, None] * torch.sin(kx * ax[2] + 0.3)[None, None, :]
    return (out * mask).reshape(-1)


def _operator(c, **opts):
    geom, h = _geometry(c)
    return dm.Operator(geom, _dims(c), h, c.get("sigma", 5.0), **opts)


MODES = {"mg64": dm.SOLVE_FGMRES_MG64, "mg32": dm.SOLVE_FGMRES_MG32, "pcg64": dm.SOLVE_PCG64}


def _weights(g):
    """Weights of the size a trained network has."""
    out = []
    for cin, cout, gain in ((10, 16, 1.0), (16, 16, 1.0), (16, 3, 0.3)):
        bound = gain * math.sqrt(6.0 / (27 * cin))
        out.append((torch.rand(27 * cin * cout, generator=g, device=DEV) * 2 - 1) * bound)
    return torch.cat(out)


def _vectors(c, seed, frac, n):
    """The face vectors that a case's call takes."""
    g, mask = _gen(seed), _active(frac, n)
    if c["kind"] == "apply":
        dt = torch.float64 if c["prec"] == 64 else torch.float32
        return [_noise(mask, g, dt) for _ in range(2)]
    if c["kind"] == "vcycle":
        dt = torch.float64 if c["prec"] == 64 else torch.float32
        return [_noise(mask, g, dt) for _ in range(c["nrhs"])]
    if c["kind"] == "batch":
        return [_noise(mask, g, torch.float32)]
    if c["kind"] == "net":
        return [_noise(mask, g)]
    return [_smooth(mask, g) for _ in range(c["nrhs"])]


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "batch":
        semi, ns = _batch_grids(c)
        b = dm.Batch([dm.ellipsoid((0.5, 0.5, 0.5), s) for s in semi], [(n, n, n) for n in ns], [1.0 / n for n in ns],
                     c["sigma"])
        c["op"] = b
        c["f"] = [_vectors(c, seed + 1000 * q, m.fractions(0), m.dims)[0] for q, m in enumerate(b.members)]
        c["x"] = [torch.zeros_like(f) for f in c["f"]]
        return c
    opts = {}
    if "nu" in c:
        opts.update(nu_pre=c["nu"], nu_post=c["nu"])
    if "restart" in c:
        opts["fgmres_restart"] = c["restart"]
    if c.get("basis32"):
        opts["krylov_basis_f32"] = 1
    op = c["op"] = _operator(c, **opts)
    if kind == "eigs":
        c["seed"] = seed
        return c
    c["f"] = _vectors(c, seed, op.fractions(0), _dims(c))
    if kind == "solve":
        c["f"] = [op.apply(dm.APPLY_A, v, torch.zeros_like(v)) for v in c["f"]]
    if kind == "net":
        c["net"] = dm.Net(seed)
        c["net"].set_weights(_weights(_gen(seed + 1)).cpu().numpy())
        c["net"].attach(op)
    c["x"] = [torch.zeros_like(f) for f in c["f"]]
    return c


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    op, kind = s["op"], s["kind"]
    if kind == "apply":
        if s["which"] == "R":
            return op.residual(s["f"][0], s["f"][1], s["x"][0])
        return op.apply(dm.APPLY_M if s["which"] == "M" else dm.APPLY_K, s["f"][0], s["x"][0])
    if kind == "vcycle":
        return [op.vcycle(s["f"][0], s["x"][0])] if s["nrhs"] == 1 else op.vcycle_block(s["f"], s["x"])
    if kind == "project":
        return [op.project(s["f"][0], s["x"][0])] if s["nrhs"] == 1 else op.project_block(s["f"], s["x"])
    if kind == "solve":
        if s["nrhs"] == 1:
            info = [op.solve(s["f"][0], s["x"][0], mode=MODES[s["mode"]], rtol=s["rtol"])]
        else:
            info = op.solve_block(s["f"], s["x"], mode=MODES[s["mode"]], rtol=s["rtol"])
        return {"x": s["x"], "status": [i["status"] for i in info]}
    if kind == "eigs":
        out = op.eigs(s["k"], tol=1e-10, seed=s["seed"], solve_mode=MODES[s["mode"]], inner_rtol=s["rtol"],
                      block=s["block"])
        return {"lam": out["lam"], "status": out["status"], "n_converged": out["n_converged"]}
    if kind == "batch":
        return op.vcycle(s["f"], s["x"])
    if s["what"] == "apply":
        return dm.net_apply(op, s["f"][0], s["x"][0])
    loss, grad = dm.net_loss_grad(op, s["f"][0], None, kind=dm.NET_LOSS_RESIDUAL)
    return {"loss": loss, "grad": grad}


def work(case):
    """Every input read once and every output written once; flops of the steps' stencils (about 60 per cell and
    application of M), of a V-cycle as its sweeps, residual and transfers on all levels, of a solve as ten V-cycles
    and products (the least that its tolerances take), of the network's convolutions."""
    c = case
    if c["kind"] == "batch":
        cells = sum(n ** 3 for n in _batch_grids(c)[1])
        return {"bytes": cells * 4 * (7 + 6), "flops": cells * 60 * 5 * 8 / 7}
    cells = c["nx"] * c["ny"] * c["nz"]
    if c["kind"] == "apply":
        return {"bytes": cells * c["prec"] // 8 * (7 + (9 if c["which"] == "R" else 6)), "flops": cells * 60}
    if c["kind"] == "vcycle":
        return {"bytes": cells * c["prec"] // 8 * (7 + 6 * c["nrhs"]),
                "flops": cells * c["nrhs"] * 60 * (2 * c["nu"] + 1) * 8 / 7}
    if c["kind"] == "project":
        return {"bytes": cells * 8 * (3 + 6 * c["nrhs"]), "flops": cells * c["nrhs"] * 14 * 10 * 6}
    if c["kind"] == "solve":
        return {"bytes": cells * 8 * (7 + 6 * c["nrhs"]),
                "flops": cells * c["nrhs"] * 60 * 10 * ((2 * c["nu"] + 1) * 8 / 7 + 1)}
    if c["kind"] == "eigs":
        return {"bytes": cells * 8 * 7, "flops": cells * c["k"] * 5 * 60 * 10 * (5 * 8 / 7 + 1)}
    mul = 1 if c["what"] == "apply" else 3
    return {"bytes": cells * 8 * 6 + cells * 14, "flops": cells * 2 * 27 * (10 * 16 + 16 * 16 + 16 * 3) * mul}


# ---------------------------------------------------------------------------
# 64-bit results from plain torch
# ---------------------------------------------------------------------------

def _sh(a, dim, by):
    """a at the neighbour `by` steps up along an axis (0 = x, 1 = y, 2 = z)."""
    return torch.roll(a, -by, -1 - dim)


class _Grid:
    """One level: fractions as padded (7, nz+2, ny+2, nx+2) blocks, and the method's steps on face vectors of shape
    (..., 3, nz+2, ny+2, nx+2)."""

    def __init__(self, frac, n, h, sigma, pmc):
        self.n, self.h, self.sigma, self.pmc = n, h, sigma, pmc
        self.a, self.l, self.v = frac[:3], frac[3:6], frac[6]
        self.vinv = torch.where(self.v > 0, 1 / self.v.clamp(min=1e-300), torch.zeros_like(self.v))
        self.act = _owned(self.a > 0)
        self.cell = _owned(self.v > 0)
        l, a, ih2 = self.l, self.a, 1 / (h * h)
        d = []
        for c in range(3):
            p, q = [(1, 2), (0, 2), (0, 1)][c]
            t = l[p] + _sh(l[p], q, 1) + l[q] + _sh(l[q], p, 1) + a[c] ** 2 * (_sh(self.vinv, c, -1) + self.vinv)
            # an edge in a symmetry plane sees a tangential face and its mirror image
            for ax, on in enumerate(pmc):
                if on and ax != c:
                    e = 3 - ax - c
                    t = t.clone()
                    t.select(-1 - ax, 1).add_(l[e].select(-1 - ax, 1))
            d.append(ih2 * t - sigma * a[c])
        self.diag = torch.stack(d)
        idx = [torch.arange(s, device=DEV) for s in self.v.shape]
        self.colour = (idx[0][:, None, None] + idx[1][None, :, None] + idx[2][None, None, :] + 1) % 2

    def mirror(self, x):
        for ax, on in enumerate(self.pmc):
            if on:
                g, lo, hi = (x.select(-1 - ax, i) for i in range(3))
                for c in range(3):
                    g[..., c, :, :] = hi[..., c, :, :] if c == ax else -lo[..., c, :, :]
        return x

    def curlcurl(self, x):
        X, Y, Z = x[..., 0, :, :, :], x[..., 1, :, :, :], x[..., 2, :, :, :]
        l = self.l
        wx = l[0] * (Z - _sh(Z, 1, -1) - Y + _sh(Y, 2, -1))
        wy = l[1] * (X - _sh(X, 2, -1) - Z + _sh(Z, 0, -1))
        wz = l[2] * (Y - _sh(Y, 0, -1) - X + _sh(X, 1, -1))
        r = torch.stack([wy - _sh(wy, 2, 1) + _sh(wz, 1, 1) - wz, -wx + _sh(wx, 2, 1) + wz - _sh(wz, 0, 1),
                         wx - _sh(wx, 1, 1) - wy + _sh(wy, 0, 1)], -4)
        return r / (self.h * self.h)

    def flux(self, x):
        ax = self.a * x
        return sum(_sh(ax[..., c, :, :, :], c, 1) - ax[..., c, :, :, :] for c in range(3))

    def graddiv(self, x):
        q = self.vinv * self.flux(x)
        return torch.stack([self.a[c] * (_sh(q, c, -1) - q) for c in range(3)], -4) / (self.h * self.h)

    def M(self, x):
        return self.mirror((self.curlcurl(x) + self.graddiv(x) - self.sigma * self.a * x) * self.act)

    def K(self, x):
        return self.mirror(self.curlcurl(x) * self.act)

    def sweep(self, f, x, reverse):
        classes = [(c, k) for c in range(3) for k in range(2)]
        for c, k in reversed(classes) if reverse else classes:
            on = self.act[c] & (self.colour == k)
            new = (f - self.M(x))[..., c, :, :, :] / self.diag[c].masked_fill(~on, 1.0)
            x[..., c, :, :, :] += torch.where(on, new, torch.zeros_like(new))
            self.mirror(x)
        return x


def _coarsen(frac, n):
    """Fractions of the next coarser grid: means of the fine ones."""
    m = tuple(v // 2 for v in n)
    out = torch.zeros((7,) + _pshape(m), device=DEV, dtype=torch.float64)
    for b in range(7):
        along = [b] if b < 3 else [a for a in range(3) if a != b - 3] if b < 6 else []   # axes sampled, not averaged
        t = frac[b][1:, 1:, 1:]
        for a in range(3):
            d = 2 - a
            if a in along:
                t = t.index_select(d, torch.arange(0, n[a] + 1, 2, device=DEV))
            else:
                k = torch.arange(0, n[a], 2, device=DEV)
                t = 0.5 * (t.index_select(d, k) + t.index_select(d, k + 1))
        out[b][1:1 + t.shape[0], 1:1 + t.shape[1], 1:1 + t.shape[2]] = t
    return out, m


def _mirror_fractions(frac, pmc):
    """Fractions beyond a symmetry plane: the mirror images of those inside."""
    for ax, on in enumerate(pmc):
        if on:
            for b in range(7):
                nodal = (b < 3 and b == ax) or (3 <= b < 6 and b - 3 != ax)
                t = frac[b]
                t.select(-1 - ax, 0).copy_(t.select(-1 - ax, 2 if nodal else 1))
    return frac


class _Cycle:
    """The geometric V-cycle."""

    def __init__(self, frac, n, h, sigma, pmc, nu):
        self.nu, self.g = nu, []
        f = torch.from_numpy(frac).to(DEV).reshape((7,) + _pshape(n)).clone()
        while True:
            self.g.append(_Grid(f, n, h, sigma, pmc))
            if any(v % 2 for v in n) or max(n) <= 8 or min(n) < 4:
                break
            f, n = _coarsen(f, n)
            _mirror_fractions(f, pmc)
            h *= 2
        g = self.g[-1]
        at = g.act.reshape(-1).nonzero()[:, 0]
        A = torch.zeros(at.numel(), at.numel(), device=DEV, dtype=torch.float64)
        for i in range(0, at.numel(), 512):
            k = at[i:i + 512]
            e = torch.zeros(k.numel(), g.act.numel(), device=DEV, dtype=torch.float64)
            e[torch.arange(k.numel(), device=DEV), k] = 1
            A[:, i:i + 512] = g.M(g.mirror(e.reshape(-1, *g.act.shape))).reshape(k.numel(), -1)[:, at].T
        self.at, self.lu = at, torch.linalg.lu_factor(A)

    def shares(self, g, c):
        """Shares of the fine faces below and above a coarse face along its normal."""
        a = g.a[c]
        return tuple(torch.where(a > 0, a / (a + _sh(a, c, d)).clamp(min=1e-300), torch.zeros_like(a)) for d in (-1, 1))

    def restrict(self, gf, gc, r):
        out = torch.zeros_like(gc.a)
        for c in range(3):
            lo, hi = self.shares(gc, c)
            t = [r[c], _sh(r[c], c, -1), _sh(r[c], c, 1)]
            for k in range(3):
                t[k] = t[k][1:-1, 1:-1, 1:-1]
                for a in range(3):
                    d = 2 - a
                    i = torch.arange(0, gf.n[a], 2, device=DEV)
                    t[k] = t[k].index_select(d, i) + (0 if a == c else t[k].index_select(d, i + 1))
            s = (slice(1, -1),) * 3
            out[c][s] = 0.125 * (t[0] + lo[s] * t[1] + hi[s] * t[2])
        return gc.mirror(out * gc.act)

    def prolong(self, gf, gc, xc):
        out = torch.zeros_like(gf.a)
        for c in range(3):
            a, x = gc.a[c], xc[c]
            up = (a * x + _sh(a, c, 1) * _sh(x, c, 1)) / (a + _sh(a, c, 1)).clamp(min=1e-300)
            t = torch.stack([x, up])[:, 1:-1, 1:-1, 1:-1]
            for ax in range(3):
                t = t.repeat_interleave(2, 3 - ax)
            odd = torch.arange(gf.n[c], device=DEV).reshape([-1 if d == 2 - c else 1 for d in range(3)]) % 2 == 1
            out[c][1:-1, 1:-1, 1:-1] = torch.where(odd, t[1], t[0])
        return gf.mirror(out * gf.act)

    def __call__(self, f, l=0):
        g = self.g[l]
        x = torch.zeros_like(f)
        if l == len(self.g) - 1:
            x.reshape(-1)[self.at] = torch.linalg.lu_solve(*self.lu, f.reshape(-1)[self.at][:, None])[:, 0]
            return g.mirror(x)
        for _ in range(self.nu):
            g.sweep(f, x, False)
        c = self.g[l + 1]
        x = x + self.prolong(g, c, self(self.restrict(g, c, g.mirror((f - g.M(x)) * g.act)), l + 1))
        for _ in range(self.nu):
            g.sweep(f, x, True)
        return x


def _gmres(A, B, f, tol=1e-13, m=40):
    """Right-preconditioned restarted GMRES, twice orthogonalised."""
    x, bn = torch.zeros_like(f), f.norm()
    for _ in range(8):
        r = f - A(x)
        beta = r.norm()
        if beta <= tol * bn:
            break
        V, Z, H = [r / beta], [], torch.zeros(m + 1, m, dtype=torch.float64)
        for j in range(m):
            Z.append(B(V[j]))
            w = A(Z[j])
            Q = torch.stack(V).reshape(j + 1, -1)
            for _ in range(2):
                h = Q @ w.reshape(-1)
                w = w - (h @ Q).reshape(w.shape)
                H[:j + 1, j] += h.cpu()
            H[j + 1, j] = w.norm().cpu()
            V.append(w / w.norm())
            rhs = torch.zeros(j + 2, 1, dtype=torch.float64)
            rhs[0] = beta.cpu()
            y = torch.linalg.lstsq(H[:j + 2, :j + 1], rhs).solution
            if (H[:j + 2, :j + 1] @ y - rhs).norm() <= 0.3 * tol * bn.cpu():
                break
        x = x + sum(float(c) * z for c, z in zip(y[:, 0], Z))
    return x


def _project(g, b):
    """b - D^T psi with D A D^T psi = D A b, by Jacobi-preconditioned conjugate gradients."""
    def S(p):
        return _odd(sum(g.a[c] * (p - _sh(p, c, -1)) + _sh(g.a[c], c, 1) * (p - _sh(p, c, 1)) for c in range(3)) * g.cell)

    def _odd(p):
        for ax, on in enumerate(g.pmc):
            if on:
                p.select(-1 - ax, 0).copy_(-p.select(-1 - ax, 1))
        return p

    own = (slice(1, -1),) * 3
    dot = lambda u, v: (u[own] * v[own]).sum()   # noqa: E731
    d = sum(g.a[c] + _sh(g.a[c], c, 1) for c in range(3))
    dinv = torch.where(g.cell & (d > 0), 1 / d.clamp(min=1e-300), torch.zeros_like(d))
    r = _odd(g.flux(b) * g.cell * g.h)
    psi, z = torch.zeros_like(r), _odd(dinv * r)
    p, rz, r0 = z.clone(), dot(r, z), dot(r, r)
    for it in range(4000):
        q = S(p)
        al = rz / dot(p, q)
        psi, r = psi + al * p, r - al * q
        z = dinv * r
        new = dot(r, z)
        p = _odd(z + (new / rz) * p)
        rz = new
        if it % 25 == 0 and float(dot(r, r)) <= 1e-30 * float(r0):
            break
    _odd(psi)
    out = torch.stack([b[c] - (_sh(psi, c, -1) - psi) / g.h for c in range(3)]) * g.act
    return g.mirror(out)


def _lowest(g, k):
    """The k smallest eigenvalues of K b = lambda A b, dense: a large grad-div penalty moves the gradients away."""
    at = g.act.reshape(-1).nonzero()[:, 0]
    s = 1 / g.a.reshape(-1)[at].sqrt()
    A = torch.zeros(at.numel(), at.numel(), device=DEV, dtype=torch.float64)
    for i in range(0, at.numel(), 512):
        j = at[i:i + 512]
        e = torch.zeros(j.numel(), g.act.numel(), device=DEV, dtype=torch.float64)
        e[torch.arange(j.numel(), device=DEV), j] = 1
        e = e.reshape(-1, *g.act.shape)
        A[:, i:i + 512] = (g.curlcurl(e) + 50 * g.graddiv(e)).reshape(j.numel(), -1)[:, at].T
    A = A * s[:, None] * s[None, :]
    L = torch.linalg.cholesky(0.5 * (A + A.T))
    Q = torch.randn(at.numel(), 3 * k + 8, generator=_gen(1), device=DEV, dtype=torch.float64)
    for _ in range(80):
        Q = torch.linalg.qr(torch.cholesky_solve(Q, L))[0]
    # Rayleigh quotients on K alone
    q = torch.zeros(Q.shape[1], g.act.numel(), device=DEV, dtype=torch.float64)
    q[:, at] = (Q * s[:, None]).T
    KQ = g.curlcurl(q.reshape(-1, *g.act.shape)).reshape(q.shape[0], -1)[:, at]
    R = q[:, at] @ KQ.T
    return torch.linalg.eigvalsh((0.5 * (R + R.T)).cpu())[:k].numpy()


def _net(w, x0, n, act):
    """The three convolutions on (nz+2, ny+2, nx+2, channels)."""
    at = 0
    for cin, cout, last in ((10, 16, False), (16, 16, False), (16, 3, True)):
        W = w[at:at + 27 * cin * cout].reshape(27, cin, cout)
        at += 27 * cin * cout
        y = 0
        for t in range(27):
            dx, dy, dz = t % 3, (t // 3) % 3, t // 9
            y = y + x0[dz:dz + n[2], dy:dy + n[1], dx:dx + n[0]] @ W[t]
        if not last:
            x0 = torch.nn.functional.pad(y.relu(), (0, 0, 1, 1, 1, 1, 1, 1))
    return torch.nn.functional.pad(y, (0, 0, 1, 1, 1, 1, 1, 1)).permute(3, 0, 1, 2) * act


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "batch":
        semi, ns = _batch_grids(c)
        out = []
        for q, (s, m) in enumerate(zip(semi, ns)):
            n = (m, m, m)
            fr = dm.compute_fractions(dm.ellipsoid((0.5, 0.5, 0.5), s), n, 1.0 / m)
            f = _vectors(c, seed + 1000 * q, fr, n)[0].double().reshape(3, *_pshape(n))
            out.append(_Cycle(fr, n, 1.0 / m, c["sigma"], (0, 0, 0), 2)(f).reshape(-1))
        return out
    if kind == "eigs" and c["nx"] * c["ny"] * c["nz"] > 5000:
        return None
    n = _dims(c)
    geom, h = _geometry(c)
    pmc = tuple(int(b == dm.BC_PMC) for b in geom.bc_lo)
    fr = dm.compute_fractions(geom, n, h)
    g = _Grid(torch.from_numpy(fr).to(DEV).reshape((7,) + _pshape(n)), n, h, c.get("sigma", 5.0), pmc)
    if kind == "eigs":
        return {"lam": _lowest(g, c["k"]), "status": None, "n_converged": None}
    vec = [g.mirror(v.double().reshape(3, *_pshape(n))) for v in _vectors(c, seed, fr, n)]
    if kind == "apply":
        f, x = vec
        return ((f - g.M(x)) * g.act if c["which"] == "R" else g.M(f) if c["which"] == "M" else g.K(f)).reshape(-1)
    if kind == "project":
        return [_project(g, v).reshape(-1) for v in vec]
    if kind == "vcycle":
        cyc = _Cycle(fr, n, h, c["sigma"], pmc, c["nu"])
        return [cyc(v).reshape(-1) for v in vec]
    if kind == "solve":
        cyc = _Cycle(fr, n, h, c["sigma"], pmc, c["nu"])
        # on the owned active faces; the mirror images beyond a symmetry plane follow from them
        A = lambda x: g.M(g.mirror(x.clone())) * g.act      # noqa: E731
        B = lambda x: cyc(g.mirror(x.clone())) * g.act      # noqa: E731
        xs = [g.mirror(_gmres(A, B, g.a * v * g.act)) for v in vec]
        return {"x": [x.reshape(-1) for x in xs], "status": [None] * len(xs)}
    w = _weights(_gen(seed + 1)).double().requires_grad_(c["what"] == "grad")
    r = vec[0]
    s = (r[g.act] ** 2).mean().sqrt()
    x0 = torch.cat([r / s, _owned(torch.cat([g.a, g.l, g.v[None]]))]).permute(1, 2, 3, 0).contiguous()
    d = _net(w, x0, n, g.act) * (s * h * h)
    if c["what"] == "apply":
        return d.reshape(-1)
    loss = ((r - g.M(d)) ** 2 * g.act).sum() / (r ** 2).sum()
    loss.backward()
    return {"loss": float(loss), "grad": w.grad.cpu().numpy()}

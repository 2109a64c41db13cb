"""Performance cases of the framework: what a simulation, an analysis script or
the training of the learned start asks of it, through the public binding
(`paper_2206_14780_amd.sph`), from a 16^3 channel to the 33.7M-particle one.

Every case is generated from its seed on the GPU: a lattice of fluid sites with
three wall layers where the geometry has them, jittered by 0.1 dp (channels of
the plane Poiseuille flow are not), the layouts and physical parameters of
`paper_2206_14780_amd.workloads`:

  channel  periodic in x and y, walls below and above          (lattice order)
  tank     walls on four sides and the bottom, open top        (random order)
  incline  periodic in x and y, wall below, open top           (random order)
  lava     periodic in x, walls below and on both y sides      (lattice order)

`exact` repeats a case in 64 bits with plain torch: it takes every particle's
neighbour candidates from its lattice site and shares nothing with the library.
"""
import math

import numpy as np
import torch

from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import warmstart as WS

LAYERS = 3                       # wall layers
TAU0, PAPA_M, MU0 = 100.0, 1000.0, 1.0  # Papanastasiou law of the incline
SLOPE = math.sin(math.radians(10.0))
F64, F32, MIXED = "f64", "f32", "mixed"
PREC = {F64: S.SPH_F64, F32: S.SPH_F32, MIXED: S.SPH_MIXED}
GEOMETRY = {  # periodic axes, walls (low, high) per axis
    "channel": ((1, 1, 0), ((0, 0), (0, 0), (1, 1))),
    "tank": ((0, 0, 0), ((1, 1), (1, 1), (1, 0))),
    "incline": ((1, 1, 0), ((0, 0), (0, 0), (1, 0))),
    "lava": ((1, 0, 0), ((0, 0), (1, 1), (1, 0))),
}
# iterations that the path needs at the listed cases' parameters (2 operator
# passes each, the conjugate gradient 1)
ITERATIONS = {"channel": 8, "tank": 68, "cg": 87, "box": 150, "lava": 60, "step": 72}


def listed():
    return [
        # the paper's Poiseuille case at dp = 1/16: the smallest solve, latency and launches
        {"name": "channel16_f64", "do": "channel", "nx": 16, "ny": 16, "nz": 16, "wall": "dynamic", "variant": "robust"},
        # one implicit step of the 1.16M tank in single precision, neighbour build included
        {"name": "tank100_f32", "do": "tank", "nx": 100, "ny": 100, "nz": 100},
        # the symmetric case on the rotated CG, odd sizes, whole step
        {"name": "cg77_f32", "do": "cg", "nx": 77, "ny": 65, "nz": 51},
        # training target of the learned start: a 64^3 box solved to full accuracy in FP64
        {"name": "box64_f64", "do": "box", "nx": 64, "ny": 64, "nz": 64},
        # the headline step: 33.7M lava channel, learned start, FP32 operator, FP64 solution
        {"name": "lava320_learned", "do": "lava", "nx": 320, "ny": 320, "nz": 320},
        # semi-implicit step of the non-Newtonian incline: two solves, advection, viscosity update
        {"name": "incline48_step", "do": "step", "nx": 48, "ny": 48, "nz": 48},
        # one product with the cached operator (residuals, monitoring), the wider Gaussian support
        {"name": "apply_gauss_f64", "do": "apply", "nx": 63, "ny": 57, "nz": 49, "prec": F64, "kernel": "gaussian",
         "jacobi": False},
        # the paper's matrix-free gemv through the allocation-free entry point
        {"name": "apply_otf_f32", "do": "otf", "nx": 60, "ny": 60, "nz": 60, "prec": F32, "kernel": "wendland",
         "jacobi": True},
        # viscosity update between solves
        {"name": "viscosity100", "do": "viscosity", "nx": 100, "ny": 100, "nz": 100, "prec": F64},
        # neighbour lists for analysis: build and canonical export
        {"name": "lists64", "do": "lists", "nx": 64, "ny": 64, "nz": 64, "kernel": "wendland"},
        # one Adam step of the learned start's training at its batch size
        {"name": "mlp_train_65536", "do": "train", "n": 65536},
        # the network on the samples of one 64^3 box
        {"name": "mlp_forward_985k", "do": "infer", "n": 984900},
    ]


def _side(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["channel", "tank", "cg", "box", "lava", "step", "apply", "otf", "viscosity", "lists", "train",
                     "infer"])
    if do == "train":
        return {"do": do, "n": _side(rng, 300, 262144)}
    if do == "infer":
        return {"do": do, "n": _side(rng, 100, 12000000)}
    lo, hi = {"channel": (8, 26), "tank": (24, 120), "cg": (20, 120), "box": (16, 72), "lava": (24, 240),
              "step": (14, 52), "apply": (16, 100), "otf": (12, 62), "viscosity": (16, 130), "lists": (12, 80)}[do]
    mid = _side(rng, lo, hi)
    c = {"do": do}
    for a in ("nx", "ny", "nz"):
        c[a] = max(lo, min(hi, int(round(mid * rng.uniform(0.75, 1.3)))))
    if do == "channel":
        c["wall"] = rng.choice(["dynamic", "dummy"])
        c["variant"] = rng.choice(["robust", "standard"])
    if do == "otf":
        while c["nx"] * c["ny"] * (c["nz"] + LAYERS) > S.SPH_NOALLOC_MAX_N:
            c["nz"] -= 1
    if do in ("apply", "otf", "lists"):
        c["kernel"] = rng.choice(["wendland", "gaussian"])
    if do in ("apply", "otf"):
        c["jacobi"] = rng.random() < 0.5
    if do in ("apply", "otf", "viscosity"):
        c["prec"] = rng.choice([F64, F32])
    return c


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo


def _smooth(g, pos, length):
    """Eight random plane waves (wavelength length/4 .. length), scaled to about [0, 1]."""
    d = torch.randn((8, 3), generator=g, device="cuda", dtype=torch.float64)
    d = d / d.norm(dim=1, keepdim=True)
    k = d * (2.0 * math.pi / _uniform(g, (8, 1), length / 4.0, length))
    ph, am = _uniform(g, (8,), 0.0, 2.0 * math.pi).tolist(), _uniform(g, (8,), 0.5, 1.0).tolist()
    out = torch.zeros_like(pos[0])
    for m, kv in enumerate(k.tolist()):
        out += am[m] * torch.cos(kv[0] * pos[0] + kv[1] * pos[1] + kv[2] * pos[2] + ph[m])
    lo, hi = out.min(), out.max()
    return (out - lo) / (hi - lo)


class Setup:
    """Lattice, particle arrays (lattice order) and the order the caller lists them in."""

    def __init__(self, geometry, n, dp, g, jitter=0.1, shuffle=True):
        self.per, self.walls = GEOMETRY[geometry]
        self.n, self.dp = n, dp
        off = [LAYERS * w[0] for w in self.walls]
        self.shape = [n[a] + LAYERS * (self.walls[a][0] + self.walls[a][1]) for a in range(3)]
        nx, ny, nz = self.shape
        self.N = nx * ny * nz
        ar = torch.arange(self.N, device="cuda", dtype=torch.int64)
        idx = [ar % nx - off[0], (ar // nx) % ny - off[1], ar // (nx * ny) - off[2]]
        fluid = torch.ones(self.N, dtype=torch.bool, device="cuda")
        for a in range(3):
            fluid &= (idx[a] >= 0) & (idx[a] < n[a])
        self.fluid = fluid
        self.pos = []
        for a in range(3):
            p = (idx[a].to(torch.float64) + 0.5) * dp
            if jitter > 0.0:
                p = p + torch.where(fluid, _uniform(g, (self.N,), -jitter * dp, jitter * dp), torch.zeros_like(p))
            self.pos.append(p)
        del idx, ar
        self.lo = [-off[a] * dp for a in range(3)]
        self.hi = [(self.shape[a] - off[a]) * dp for a in range(3)]
        self.h = 1.3 * dp
        self.rho = torch.ones(self.N, dtype=torch.float64, device="cuda")
        self.mass = self.rho * dp ** 3
        self.perm = torch.randperm(self.N, generator=g, device="cuda") if shuffle else None

    def listed(self, a):
        """The array in the caller's order."""
        return a.contiguous() if self.perm is None else a[self.perm].contiguous()

    def particles(self, mu):
        t = self.listed
        return S.Particles(*[t(p) for p in self.pos], t(self.mass), t(self.rho), t(mu),
                           t(torch.where(self.fluid, 0, 1).to(torch.uint8)))

    def domain(self, kernel="wendland"):
        return S.make_domain(self.lo, self.hi, self.per, self.h,
                             S.SPH_KERNEL_GAUSSIAN if kernel == "gaussian" else S.SPH_KERNEL_WENDLAND)

    def velocity(self, g, noise, amp=1.0):
        """A smooth field per component plus noise on fluid rows, 0 on wall rows."""
        L = float(max(self.n)) * self.dp
        out = []
        for _ in range(3):
            u = amp * (2.0 * _smooth(g, self.pos, L) - 1.0)
            u = u + noise * torch.randn(self.N, generator=g, device="cuda", dtype=torch.float64)
            out.append(torch.where(self.fluid, u, torch.zeros_like(u)))
        return out

    def vary(self, g):
        """Densities and masses that differ from particle to particle by a few percent."""
        self.rho = _uniform(g, (self.N,), 0.95, 1.05)
        self.mass = self.rho * self.dp ** 3 * _uniform(g, (self.N,), 0.97, 1.03)


def _papa(D):
    safe = torch.where(D > 0.0, D, torch.ones_like(D))
    return TAU0 * torch.where(D > 0.0, -torch.expm1(-PAPA_M * safe) / safe, torch.full_like(D, PAPA_M)) + MU0


def _inputs(case, seed):
    """The system of a case: its arrays in lattice order and its parameters."""
    g = _gen(seed)
    do, n = case["do"], tuple(case[a] for a in ("nx", "ny", "nz"))
    q = {"wall": "dummy", "avg": "arith", "jacobi": True, "kernel": "wendland", "variant": "robust", "prec": F64,
         "tol": 1e-6}
    if do == "channel":
        dp = 1.0 / n[2]
        s = Setup("channel", n, dp, g, jitter=0.0, shuffle=False)
        nu = float(10.0 ** _uniform(g, (1,), -0.5, 0.5))
        mu = nu * s.rho
        dt = 10.0 * dp * dp / nu
        # a body force along x, and a little across it, so that the three components differ
        f = [dt * float(v) for v in _uniform(g, (3,), 0.2, 1.0)]
        rhs = [torch.where(s.fluid, torch.full_like(mu, v), torch.zeros_like(mu)) for v in f]
        q.update(wall=case["wall"], variant=case["variant"], tol=1e-8)
        u = None
    elif do in ("tank", "cg"):
        s = Setup("tank", n, 1.0, g)
        nu = 10.0
        mu, dt = nu * s.rho, 50.0 / nu
        rhs = [torch.where(s.fluid, 0.1 * torch.randn(s.N, generator=g, device="cuda", dtype=torch.float64),
                           torch.zeros_like(mu)).to(torch.float32).to(torch.float64) for _ in range(3)]
        u = rhs
        q.update(prec=F32)
        if do == "cg":
            q.update(wall="dynamic", variant="cg")
    elif do == "box":
        s = Setup("tank", n, 1.0, g)
        nu = float(10.0 ** _uniform(g, (1,), 0.0, 3.0))
        mu, dt = nu * s.rho, float(_uniform(g, (1,), 10.0, 100.0)) / nu
        rhs = u = s.velocity(g, 0.1)
        q.update(tol=1e-12)
    elif do == "lava":
        s = Setup("lava", n, 1.0, g, shuffle=False)
        T = 1000.0 + 200.0 * _smooth(g, s.pos, float(max(n)))
        mu = 1e4 * torch.exp(-0.02 * T)
        dt = 50.0 / (1e4 * math.exp(-20.0))
        # the velocity some steps after rest: the drive accumulated over a smooth profile
        u = s.velocity(g, 0.0, amp=0.05)
        prof = torch.clamp(s.pos[2] / n[2], 0.0, 1.0) * torch.clamp(s.pos[1] / n[1] * (1.0 - s.pos[1] / n[1]), min=0.0)
        u[0] = torch.where(s.fluid, u[0] + 8.0 * SLOPE * prof, torch.zeros_like(prof))
        rhs = [torch.where(s.fluid, u[c] + (SLOPE if c == 0 else 0.0), torch.zeros_like(u[c])) for c in range(3)]
        q.update(avg="harmonic", prec=MIXED)
    elif do == "step":
        s = Setup("incline", n, 1.0, g)
        mu = _papa(_smooth(g, s.pos, float(max(n))))
        dt = 20.0 * 50.0 / (PAPA_M * TAU0 + MU0)
        u = s.velocity(g, 0.0, amp=4.0)
        rhs = None
        q.update(avg="harmonic", tol=1e-12)
    else:  # products, viscosity update and lists: the incline with uneven particles
        # lists: one set of positions, listed in another order by every seed
        s = Setup("incline", n, 1.0, _gen(3) if do == "lists" else g)
        if do == "lists":
            s.perm = torch.randperm(s.N, generator=g, device="cuda")
        s.vary(g)
        mu = _papa(_smooth(g, s.pos, float(max(n))))
        dt = 50.0 / (PAPA_M * TAU0 + MU0)
        u = s.velocity(g, 0.05)
        rhs = None
        for k in ("prec", "kernel", "jacobi"):
            q[k] = case.get(k, q[k])
        q.update(avg="harmonic")
        if q["prec"] == F32:
            u = [v.to(torch.float32).to(torch.float64) for v in u]
    return s, mu, dt, u, rhs, q


def _mlp_inputs(case, seed, pool):
    g = _gen(seed)
    smp = torch.randn((pool, S.SPH_MLP_SAMPLE), generator=g, device="cuda", dtype=torch.float32)
    # features (u/U, d/U, relative log10 nu, log10 stiffness), basis (b, u, d)/U, target V/U
    smp[:, 2] *= 0.3
    smp[:, 3] = smp[:, 3].abs() + 0.5
    smp[:, 5] = smp[:, 0]
    smp[:, 6] = smp[:, 1]
    smp[:, 7] = 0.5 * smp[:, 4] + 0.3 * smp[:, 5] + 0.1 * smp[:, 6]
    return g, smp, torch.from_numpy(WS.load()).cuda()


_context = []


def _ctx():
    """The one context of the program (workspaces and stream binding)."""
    if not _context:
        _context.append(S.Context(0))
    return _context[0]


def prepare(case, seed):
    do, ctx = case["do"], _ctx()
    if do == "infer":
        _, smp, w = _mlp_inputs(case, seed, case["n"])
        return {"do": do, "ctx": ctx, "n": case["n"], "samples": smp, "weights": w}
    if do == "train":
        # halfway through a training: moments of some size
        g, smp, w = _mlp_inputs(case, seed, 1 << 20)
        m = 1e-3 * torch.randn(S.SPH_MLP_NPARAM, generator=g, device="cuda", dtype=torch.float32)
        v = 1e-5 + 1e-4 * torch.rand(S.SPH_MLP_NPARAM, generator=g, device="cuda", dtype=torch.float32)
        idx = torch.randint(0, 1 << 20, (case["n"],), generator=g, device="cuda", dtype=torch.int32)
        return {"do": do, "ctx": ctx, "n": case["n"], "samples": smp, "weights": w, "m": m, "v": v, "idx": idx}
    s, mu, dt, u, rhs, q = _inputs(case, seed)
    vec = torch.float32 if q["prec"] == F32 else torch.float64
    st = {"do": do, "ctx": ctx, "prec": PREC[q["prec"]], "parts": s.particles(mu), "dom": s.domain(q["kernel"])}
    op = S.SPH_OP_ONTHEFLY if do == "otf" else S.SPH_OP_CACHED
    st["params"] = S.make_params(dt, S.SPH_WALL_DYNAMIC if q["wall"] == "dynamic" else S.SPH_WALL_DUMMY,
                                 S.SPH_AVG_HARMONIC if q["avg"] == "harmonic" else S.SPH_AVG_ARITH, q["jacobi"], op)
    if u is not None:
        st["u"] = [s.listed(a).to(vec) for a in u]
    if rhs is not None:
        st["rhs"] = [s.listed(a).to(vec) for a in rhs]
        if do == "lava":
            st["warm"] = torch.from_numpy(WS.load()).cuda()
        st["opts"] = S.make_opts(tol=q["tol"], x0_given=u is not None, warm_params=st.get("warm"),
                                 variant={"robust": S.SPH_ROBUST, "standard": S.SPH_STANDARD, "cg": S.SPH_CG}[q["variant"]])
    if do == "step":
        st["opts"] = S.make_opts(tol=q["tol"])
        st["step"] = S.make_step_params((SLOPE, 0.0, 0.0), (TAU0, PAPA_M, MU0))
    if do in ("apply", "otf", "viscosity"):  # positions do not change between such calls
        st["nb"] = ctx.sph_build_neighbors(st["parts"], st["dom"])
    return st


def run(st):
    do, ctx = st["do"], st["ctx"]
    if do == "infer":
        out = torch.empty((st["n"], 4), dtype=torch.float32, device="cuda")
        ctx.sph_mlp_forward(st["samples"], st["n"], st["weights"], out)
        return {"out": out}
    if do == "train":
        w, m, v = st["weights"].clone(), st["m"].clone(), st["v"].clone()
        ctx.sph_mlp_train_step(st["samples"], st["idx"], st["n"], w, m, v, 500, 1e-3, want_loss=False)
        return {"weights": w, "m": m, "v": v}
    p = st["parts"]
    if do == "lists":
        nb = ctx.sph_build_neighbors(p, st["dom"])
        row_ptr, cols = ctx.sph_neighbors_export(nb)
        nb.free()
        return {"row_ptr": row_ptr, "cols": cols}
    if do == "viscosity":
        mu, shear = torch.empty_like(p.mu), torch.empty_like(p.mu)
        ctx.sph_visc_papanastasiou(st["nb"], p, st["prec"], st["u"], TAU0, PAPA_M, MU0, mu, shear)
        return {"mu": mu, "shear": shear}
    if do in ("apply", "otf"):
        y = [torch.empty_like(t) for t in st["u"]]
        f = ctx.sph_visc_apply if do == "apply" else ctx.sph_visc_apply_noalloc
        f(st["nb"], p, st["params"], st["prec"], st["u"], y)
        return {"y": y}
    if do == "step":
        pos, u, mu = [torch.empty_like(p.x) for _ in range(3)], [t.clone() for t in st["u"]], torch.empty_like(p.mu)
        ctx.sph_semi_implicit_step(st["dom"], p, st["params"], st["prec"], st["step"], st["opts"], pos, u, mu)
        return {"pos": pos, "u": u, "mu": mu}
    # one implicit step: neighbour lists at the current positions, then the solve
    x = [t.clone() for t in st["u"]] if "u" in st else [torch.empty_like(t) for t in st["rhs"]]
    nb = ctx.sph_build_neighbors(p, st["dom"])
    ctx.sph_visc_solve(nb, None, p, st["params"], st["prec"], st["rhs"], x, st["opts"])
    nb.free()
    return {"x": x}


def work(case):
    """Bytes and operations of one pass: every array of the call once, and for a solve or a product with
    the cached operator the matrix (a value and a 16-bit column step per entry) once per operator pass,
    with the row's operand and result vectors."""
    do = case["do"]
    if do == "infer":
        return {"bytes": 48 * case["n"], "flops": 2 * (4 * 64 + 2 * 64 * 64 + 64 * 3) * case["n"]}
    if do == "train":
        return {"bytes": 36 * case["n"] + 24 * S.SPH_MLP_NPARAM, "flops": 6 * (4 * 64 + 2 * 64 * 64 + 64 * 3) * case["n"]}
    geo = {"channel": "channel", "tank": "tank", "cg": "tank", "box": "tank", "lava": "lava"}.get(do, "incline")
    n = 1.0
    for a, k in enumerate(("nx", "ny", "nz")):
        n *= case[k] + LAYERS * sum(GEOMETRY[geo][1][a])
    pairs = (250 if case.get("kernel") == "gaussian" else 80) * n
    props = 57.0  # positions, mass, rho, mu, type
    elt = 4 if do in ("tank", "cg", "lava") or case.get("prec") == F32 else 8
    if do == "lists":
        return {"bytes": 24 * n + 8 * n + 4 * pairs, "flops": 8 * pairs}
    if do == "viscosity":
        return {"bytes": n * (props + 3 * elt + 16), "flops": 40 * pairs}
    if do == "otf":
        return {"bytes": n * (props + 6 * elt), "flops": 30 * pairs}
    if do == "apply":
        return {"bytes": n * (props + 6 * elt) + 2 * pairs * (elt + 2), "flops": 36 * pairs}
    its = ITERATIONS[do]
    passes = its * (1 if do == "cg" else 2)
    return {"bytes": n * (props + 9 * 8) + passes * (pairs * (elt + 2) + n * 6 * elt), "flops": passes * 9 * pairs}


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------
class Pairs:
    """Neighbours of every particle of a Setup at positions `pos`: idx (N, K) with N for none, r (N, K, 3)
    displacements r_row - r_idx by minimum image, r2 (N, K)."""

    def __init__(self, s, pos, kernel):
        self.s, self.N, self.kernel = s, s.N, kernel
        cut = (3.0 if kernel == "gaussian" else 2.0) * s.h
        reach = cut / s.dp + 0.6
        m = int(math.ceil(reach))
        offs = [(i, j, k) for k in range(-m, m + 1) for j in range(-m, m + 1) for i in range(-m, m + 1)
                if (i, j, k) != (0, 0, 0) and i * i + j * j + k * k <= reach * reach]
        nx, ny, nz = s.shape
        ar = torch.arange(s.N, device="cuda")
        ijk = [ar % nx, (ar // nx) % ny, ar // (nx * ny)]
        P = torch.stack(pos, dim=1)
        P = torch.cat([P, torch.full((1, 3), 1e300, dtype=torch.float64, device="cuda")])
        period = [(s.hi[a] - s.lo[a]) if s.per[a] else 0.0 for a in range(3)]
        idx = []
        for o in offs:
            ok = torch.ones(s.N, dtype=torch.bool, device="cuda")
            c = []
            for a in range(3):
                v = ijk[a] + o[a]
                if s.per[a]:
                    v = v % s.shape[a]
                else:
                    ok &= (v >= 0) & (v < s.shape[a])
                c.append(v)
            t = torch.where(ok, (c[2] * ny + c[1]) * nx + c[0], s.N)
            d = self._disp(P[:s.N] - P[t], period)
            r2 = d.square().sum(1)
            near = ok & (r2 < cut * cut)
            idx.append(torch.where(near, t, s.N).to(torch.int32))
        idx = torch.stack(idx, 1)
        # neighbours first, the width of the longest row
        order = torch.sort((idx == s.N).to(torch.uint8), dim=1, stable=True).indices
        k = int((idx < s.N).sum(1).max())
        self.idx = torch.gather(idx, 1, order[:, :k]).long()
        self.on = self.idx < s.N
        self.period = period
        self.P = P

    @staticmethod
    def _disp(d, period):
        for a in range(3):
            if period[a]:
                d[..., a] -= period[a] * torch.round(d[..., a] / period[a])
        return d

    def rows(self):
        step = max(1, (1 << 26) // max(1, self.idx.shape[1]))
        for b in range(0, self.N, step):
            yield slice(b, min(self.N, b + step))

    def geometry(self, r):
        """Displacements and q of the pairs of rows r."""
        i = self.idx[r]
        d = self._disp(self.P[:self.N][r][:, None, :] - self.P[i], self.period)
        d = torch.where(self.on[r][..., None], d, torch.zeros_like(d))
        return i, d, d.square().sum(-1).sqrt() / self.s.h

    def F(self, q, on):
        h5 = self.s.h ** 5
        if self.kernel == "gaussian":
            f = -2.0 * torch.exp(-q * q) / self._norm()
        else:
            f = 105.0 / (128.0 * math.pi) * (q - 2.0) ** 3
        return torch.where(on, f / h5, torch.zeros_like(f))

    def W(self, q, on):
        if self.kernel == "gaussian":
            w = (torch.exp(-q * q) - math.exp(-9.0)) / self._norm()
        else:
            w = 21.0 / (16.0 * math.pi) * (1.0 - 0.5 * q) ** 4 * (2.0 * q + 1.0)
        return torch.where(on, w / self.s.h ** 3, torch.zeros_like(w))

    @staticmethod
    def _norm():
        return math.pi ** 1.5 * math.erf(3.0) - 2.0 * math.pi / 3.0 * math.exp(-9.0) * 3.0 * 21.0


def _pad(a):
    return torch.cat([a, torch.ones((1,) + a.shape[1:], dtype=a.dtype, device=a.device)])


class Operator:
    """A(dt) of a Setup in difference form: A x = rs x + sum c (x_a - x)."""

    def __init__(self, s, pairs, mu, dt, q):
        self.pairs = pairs
        self.c = torch.zeros(pairs.idx.shape, dtype=torch.float64, device="cuda")
        self.D = torch.ones(s.N, dtype=torch.float64, device="cuda")
        self.rs = torch.ones_like(self.D)
        MU, RHO, M, FL = _pad(mu), _pad(s.rho), _pad(s.mass), torch.cat([s.fluid, s.fluid.new_zeros(1)])
        for r in pairs.rows():
            i, _, qq = pairs.geometry(r)
            on = pairs.on[r]
            a, b = MU[i], mu[r][:, None]
            mean2 = 4.0 * (a * b) / (a + b) if q["avg"] == "harmonic" else a + b
            w = -mean2 * M[i] * pairs.F(qq, on) / (RHO[i] * s.rho[r][:, None])
            fl = s.fluid[r]
            W = pairs.W(qq, on & FL[i]) if q["wall"] == "dummy" else torch.zeros_like(w)
            sW = W.sum(1)
            self.D[r] = torch.where(fl, 1.0 + dt * w.sum(1), torch.ones_like(sW))
            self.c[r] = torch.where(fl[:, None], -dt * w, W / torch.where(sW > 0, sW, torch.ones_like(sW))[:, None])
            self.rs[r] = torch.where(fl | ~(sW > 0), torch.ones_like(sW), torch.full_like(sW, 2.0))

    def __call__(self, x):
        y = torch.empty_like(x)
        X = _pad(x)
        step = max(1, (1 << 25) // max(1, self.c.shape[1]))
        for b in range(0, x.shape[0], step):
            r = slice(b, min(x.shape[0], b + step))
            d = X[self.pairs.idx[r]] - x[r][:, None, :]
            y[r] = self.rs[r][:, None] * x[r] + torch.bmm(self.c[r][:, None, :], d)[:, 0, :]
        return y

    def solve(self, b, x):
        """BiCGSTAB on the scaled system, restarted from the true residual until that no longer falls."""
        Di = (1.0 / self.D)[:, None]
        bb = b * Di
        nb = bb.norm(dim=0).clamp_min(1e-300)
        best, left = None, 900
        while left > 0:
            r = bb - Di * self(x)
            rel = float((r.norm(dim=0) / nb).max())
            if rel < 2e-14 or (best is not None and rel > 0.3 * best[0]):
                return x if best is None or rel < best[0] else best[1]
            best = (rel, x.clone())
            h, p, goal = r.clone(), r.clone(), 1e-4 * r.norm(dim=0)
            rho = (h * r).sum(0)
            for _ in range(200):
                left -= 1
                v = Di * self(p)
                al = self._safe(rho, (h * v).sum(0))
                s = r - al * v
                t = Di * self(s)
                om = self._safe((s * t).sum(0), (t * t).sum(0))
                x = x + al * p + om * s
                r = s - om * t
                if bool((r.norm(dim=0) <= goal).all()) or left <= 0:
                    break
                new = (h * r).sum(0)
                p = r + self._safe(new, rho) * self._safe(al, om) * (p - om * v)
                rho = new
        return x

    @staticmethod
    def _safe(a, b):
        return torch.where(b != 0, a / torch.where(b != 0, b, torch.ones_like(b)), torch.zeros_like(a))


def _viscosity(s, pairs, mu, u):
    """Viscosity and shear rate of the velocity u (N, 3)."""
    D = torch.empty(s.N, dtype=torch.float64, device="cuda")
    U, V = _pad(u), _pad(s.mass / s.rho)
    for r in pairs.rows():
        i, d, qq = pairs.geometry(r)
        vf = V[i] * pairs.F(qq, pairs.on[r])
        G = torch.bmm((vf[..., None] * -d).transpose(1, 2).contiguous(), (U[i] - u[r][:, None, :]).contiguous())
        G = 0.5 * (G + G.transpose(1, 2))
        D[r] = (2.0 * G.square().sum((1, 2))).sqrt()
    x = PAPA_M * D
    t = torch.ones_like(x)
    for k in range(8, 1, -1):
        t = 1.0 - x / k * t
    y = torch.where(x >= (362880.0 * 2.0 ** -23) ** 0.125, (1.0 - torch.exp(-x)) / torch.where(D > 0, D, torch.ones_like(D)),
                    PAPA_M * t)
    return torch.where(s.fluid, TAU0 * y + MU0, mu), D


def _exact_step(s, mu, dt, u, q):
    fl, u = s.fluid[:, None], torch.stack(u, 1)
    force = torch.tensor([SLOPE, 0.0, 0.0], dtype=torch.float64, device="cuda")
    period = [(s.hi[a] - s.lo[a]) if s.per[a] else 0.0 for a in range(3)]

    def moved(d):
        out = []
        for a in range(3):
            x = torch.where(s.fluid, s.pos[a] + d[:, a], s.pos[a])
            out.append(torch.where(s.fluid, s.lo[a] + torch.remainder(x - s.lo[a], period[a]), x) if period[a] else x)
        return out

    A = Operator(s, Pairs(s, s.pos, "wendland"), mu, 0.5 * dt, q)
    h = torch.where(fl, A.solve(torch.where(fl, u + 0.5 * dt * force, 2.0 * u), u), u)
    del A
    p1 = Pairs(s, moved(0.5 * dt * u), "wendland")
    mu1, _ = _viscosity(s, p1, mu, h)
    A = Operator(s, p1, mu1, dt, q)
    v = torch.where(fl, A.solve(torch.where(fl, u + dt * force, 2.0 * u), h), u)
    del A, p1
    pos = moved(0.5 * dt * (u + v))
    mu2, _ = _viscosity(s, Pairs(s, pos, "wendland"), mu, v)
    return pos, [v[:, c] for c in range(3)], mu2


def _mlp64(smp, w, grad):
    """Outputs (o, pred) in 64 bits with the weights as the products take them (rounded to bfloat16)."""
    shapes, parts, k = [(4, 64), (64, 64), (64, 64), (64, 3)], [], 0
    for fi, fo in shapes:
        W = w[k:k + fi * fo].to(torch.bfloat16).double().reshape(fi, fo).requires_grad_(grad)
        b = w[k + fi * fo:k + fi * fo + fo].double().requires_grad_(grad)
        parts += [W, b]
        k += fi * fo + fo
    x = smp.double()
    z = x[:, :4]
    for j in range(4):
        z = z @ parts[2 * j] + parts[2 * j + 1]
        z = torch.relu(z) if j < 3 else z
    return parts, z, (z * x[:, 4:7]).sum(1), x[:, 7]


def exact(case, seed):
    do = case["do"]
    if do == "infer":
        _, smp, w = _mlp_inputs(case, seed, case["n"])
        outs = []
        for b in range(0, case["n"], 1 << 20):
            _, o, pred, _ = _mlp64(smp[b:b + (1 << 20)], w, False)
            outs.append(torch.cat([o, pred[:, None]], 1))
        return {"out": torch.cat(outs)}
    if do == "train":
        st = prepare(case, seed)
        parts, _, pred, t = _mlp64(st["samples"][st["idx"].long()], st["weights"], True)
        (pred - t).square().mean().backward()
        g = torch.cat([p.grad.reshape(-1) for p in parts])
        m = 0.9 * st["m"].double() + 0.1 * g
        v = 0.999 * st["v"].double() + 0.001 * g * g
        step = (m / (1.0 - 0.9 ** 500)) / ((v / (1.0 - 0.999 ** 500)).sqrt() + 1e-8)
        return {"weights": st["weights"].double() - 1e-3 * step, "m": m, "v": v}
    cells = case["nx"] * case["ny"] * case["nz"]
    if do == "lists" or cells > (400000 if case.get("kernel") == "gaussian" else 1300000):
        return None
    s, mu, dt, u, rhs, q = _inputs(case, seed)
    if do == "step":
        pos, v, mu2 = _exact_step(s, mu, dt, u, q)
        return {"pos": [s.listed(p) for p in pos], "u": [s.listed(a) for a in v], "mu": s.listed(mu2)}
    pairs = Pairs(s, s.pos, q["kernel"])
    if do == "viscosity":
        m2, D = _viscosity(s, pairs, mu, torch.stack(u, 1))
        return {"mu": s.listed(m2), "shear": s.listed(D)}
    A = Operator(s, pairs, mu, dt, q)
    if do in ("apply", "otf"):
        y = A(torch.stack(u, 1))
        if q["jacobi"]:
            y = y / A.D[:, None]
        return {"y": [s.listed(y[:, c]) for c in range(3)]}
    b = torch.stack(rhs, 1)
    x = A.solve(b, torch.zeros_like(b) if u is None else torch.stack(u, 1))
    return {"x": [s.listed(x[:, c]) for c in range(3)]}

"""The work that programs have this library do, as a list of cases to time.

Each case goes through the public entry points (``Context`` and ``rollout``)
on seeded synthetic states made on the GPU: turbulent periodic boxes, the
Orszag-Tang start and noisy isothermal atmospheres between closed walls.
``exact`` evaluates the same right-hand side, step, projection or gradient
in plain float64 torch.
"""
import math

import torch

OPTIONS = ("cool", "cori", "ediffav", "lnp", "divb", "smag", "max5", "quench", "order2")
GHOST = 5                                   # ghost planes per closed wall
# eq. tconst of the scheme, as printed
RK_ALPHA, RK_BETA = (0.0, -0.641874, -1.31021), (0.46173, 0.924087, 0.390614)
# operations of one right-hand side per cell (counted on a plain evaluation)
RHS_FLOPS = 1430


# ---------------------------------------------------------------------------
# the cases
def _case(name, kind, nx, ny=None, nz=None, state="turbulent", dtype="float32", terms="core", **more):
    c = dict(kind=kind, state=state, nx=nx, ny=ny or nx, nz=nz or nx, dtype=dtype, terms=terms,
             stretch=False, tuned=False, steps=1, ncheck=0, boxes="")
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a program with its own integrator on a small ragged test box:
        # the latency of one right-hand side
        _case("rhs_20x22x24_f64", "rhs", 20, 22, 24, dtype="float64"),
        # the small Orszag-Tang run, ten steps to a call
        _case("step_orszag32_f64", "step", 32, state="orszag", dtype="float64", steps=10),
        # one step of a medium box, with the launch a context starts with
        _case("step_turb128_f32", "step", 128),
        # own integrator with a monitor: dF and the reductions that bound its dt
        _case("monitor_turb256_f32", "monitor", 256),
        # the production run: 512^3 atmosphere, tuned launch
        _case("step_strat512_f32", "step", 512, state="stratified", tuned=True),
        # float64 production at odd sizes, with the launch a context starts with
        _case("step_strat_200x180x215_f64", "step", 200, 180, 215, state="stratified", dtype="float64"),
        # every optional term on a stretched axis
        _case("step_options_150x132x140_f32", "step", 150, 132, 140, state="stratified",
              terms="+".join(OPTIONS), stretch=True),
        # 96 uneven boxes in one context, tuned launch
        _case("ensemble96_f32", "step", 0, tuned=True, boxes="48,64,80,96*24"),
        # B projected onto its solenoidal part
        _case("clean_turb256_f32", "clean", 256),
        # one adjoint step of the differentiable workload
        _case("adjoint_turb128_f32", "adjoint", 128),
        # one adjoint step with walls and every optional term
        _case("adjoint_options64_f32", "adjoint", 64, state="stratified", terms="+".join(OPTIONS)),
        # a loss through a checkpointed rollout: states and gradients
        _case("rollout_turb48_f64", "rollout", 48, dtype="float64", steps=6, ncheck=2),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "rhs", "monitor", "clean", "adjoint", "rollout", "ensemble"))
    dtype = rng.choice(("float32", "float32", "float64"))
    if kind == "ensemble":
        sizes = sorted({rng.randrange(12, 97) for _ in range(rng.randrange(2, 5))})
        return _case(None, "step", 0, dtype=dtype, boxes="%s*%d" % (",".join(map(str, sizes)), rng.randrange(2, 17)))
    lo, hi = {"step": (12, 300), "rhs": (12, 300), "monitor": (16, 300), "clean": (12, 256),
              "adjoint": (12, 120), "rollout": (12, 48)}[kind]
    n = [_size(rng, lo, hi) for _ in range(3)]
    if kind == "clean":     # transform lengths: even, as the configurations have them
        n = [max(12, 4 * (v // 4)) for v in n]
    state = "turbulent" if kind in ("clean", "rollout") else rng.choice(("turbulent", "stratified"))
    terms = "core"
    if kind in ("step", "adjoint", "rhs"):
        some = [o for o in OPTIONS if rng.random() < 0.4 and o != "order2"]
        if rng.random() < 0.4 and some:
            terms = "+".join(some)
    return _case(None, kind, n[0], n[1], n[2], state=state, dtype=dtype, terms=terms,
                 stretch=state == "stratified" and rng.random() < 0.3,
                 steps=rng.randrange(2, 6) if kind == "rollout" else (rng.choice((1, 1, 4)) if kind == "step" else 1),
                 ncheck=rng.randrange(0, 4) if kind == "rollout" else 0)


# ---------------------------------------------------------------------------
# boxes, parameters and states
def _cubes(case):
    """The box edges of an ensemble, sizes interleaved."""
    sizes, per = case["boxes"].split("*")
    return [int(s) for _ in range(int(per)) for s in sizes.split(",")]


def _boxes(case):
    if case["boxes"]:
        return [dict(nx=n, ny=n, nz=n, ngz=0, wall=False, Lx=1.0, Ly=1.0, Lz=1.0) for n in _cubes(case)]
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["state"] != "stratified":
        return [dict(nx=nx, ny=ny, nz=nz, ngz=0, wall=False, Lx=1.0, Ly=1.0, Lz=1.0)]
    b = dict(nx=nx, ny=ny, nz=nz, ngz=GHOST, wall=True, Lx=nx / nz, Ly=ny / nz, Lz=1.0)
    if case["stretch"]:
        b["zc"] = tuple(_height((k - GHOST + 0.5) / nz) for k in range(nz + 2 * GHOST))
    return [b]


def _height(u):
    """Height of a stretched axis: spacing 1.35 of the mean below, 0.85 above."""
    return u + 0.35 * u * (1.0 - u) - 0.2 * u * u * (1.0 - u)


def _options(case):
    return () if case["terms"] == "core" else tuple(case["terms"].split("+"))


def _params(case):
    p = dict(gamma=5.0 / 3.0, mu=1.0, gz=4.0 if case["state"] == "stratified" else 0.0, nu1=0.02, nu2=1.0,
             nu3=0.02, nuE=1.0, nuB=1.0, c1=0.0, Cdt=0.3, Cdtd=0.7, Cdtr=0.1)
    p.update(e_cool=1.5, t_cool=0.1, rho_cool=math.exp(-2.0), cool_cut=1, omega=(0.0, 0.5, math.sqrt(0.75)),
             c_divb=0.05, c_smag=0.15, q_max=8.0, q_lim=2.0, d2_lim=0.3)
    return p


def _dt(case):
    """A fixed stable step for the gradients."""
    b = _boxes(case)[0]
    return 0.05 * min(b["Lx"] / b["nx"], b["Ly"] / b["ny"], b["Lz"] / b["nz"])


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _shifted(n, L, face, dev):
    return (torch.arange(n, device=dev, dtype=torch.float64) + (0.0 if face else 0.5)) * (L / n)


def _orszag(b, gen, dev):
    n, tw = b["nx"], 2.0 * math.pi
    ph = torch.rand(3, generator=gen, device=dev, dtype=torch.float64)
    x = _shifted(n, 1.0, False, dev)
    shape, r0, p0 = (n, n, n), 25.0 / (36.0 * math.pi), 5.0 / (12.0 * math.pi)
    s = lambda v, ax: v.view([n if a == ax else 1 for a in range(3)]).expand(shape)   # noqa: E731
    full = lambda v: torch.full(shape, v, device=dev, dtype=torch.float64)            # noqa: E731
    u = (-torch.sin(tw * (x + ph[1])), torch.sin(tw * (x + ph[2])), torch.sin(tw * (x + ph[0])))
    return [full(r0), s(r0 * u[0], 1), s(r0 * u[1], 0), s(r0 * u[2], 2), full(1.5 * p0),
            s(u[0], 1), s(torch.sin(2 * tw * (x + ph[2])), 0), s(-u[2], 2)]


def _spectral(b, slope, gen, dev):
    """A random solenoidal vector field on 1 <= |k| <= 8 at the lower faces."""
    n = (b["nz"], b["ny"], b["nx"])
    k = torch.meshgrid(*[torch.fft.fftfreq(m, d=1.0 / m, device=dev, dtype=torch.float64) for m in n], indexing="ij")
    k = (k[2], k[1], k[0])
    kk = (k[0] ** 2 + k[1] ** 2 + k[2] ** 2).sqrt()
    amp = torch.where((kk >= 1) & (kk <= 8), kk.clamp(min=1.0) ** slope, torch.zeros_like(kk))
    s = [torch.complex(torch.randn(n, generator=gen, device=dev, dtype=torch.float64),
                       torch.randn(n, generator=gen, device=dev, dtype=torch.float64)) * amp for _ in range(3)]
    div = (k[0] * s[0] + k[1] * s[1] + k[2] * s[2]) / kk.clamp(min=1.0) ** 2
    out = []
    for a, m in enumerate((b["nx"], b["ny"], b["nz"])):
        v = (s[a] - k[a] * div) * torch.exp(-1j * math.pi * k[a] / m)
        out.append(torch.fft.ifftn(v).real)
    return out


def _turbulent(b, gen, dev):
    """rms Mach 0.5, plasma beta 1, density noise of 1 %."""
    n = (b["nz"], b["ny"], b["nx"])
    u, m = _spectral(b, -2.0, gen, dev), _spectral(b, -2.0, gen, dev)
    rms = lambda v: sum((c * c).mean() for c in v).sqrt()                             # noqa: E731
    u = [c * (0.5 / rms(u)) for c in u]
    m = [c * (math.sqrt(1.2) / rms(m)) for c in m]
    rho = 1.0 + 0.01 * torch.randn(n, generator=gen, device=dev, dtype=torch.float64)
    return [rho] + [rho * c for c in u] + [torch.full(n, 0.9, device=dev, dtype=torch.float64)] + m


def _stratified(b, gen, dev):
    """Four scale heights at rest plus noise: 1 % on rho and e, 5 % of the
    sound speed on u, a vertical field (beta 100 at mid-height) with 10 %
    horizontal parts."""
    nz, shape = b["nz"], (b["nz"] + 2 * GHOST, b["ny"], b["nx"])
    at = _height if b.get("zc") else (lambda u: u)
    col = lambda off: torch.tensor([math.exp(-4.0 * at((k - GHOST + off) / nz)) for k in range(shape[0])],   # noqa: E731
                                   device=dev, dtype=torch.float64).view(-1, 1, 1)
    noise = lambda s: s * torch.randn(shape, generator=gen, device=dev, dtype=torch.float64)                # noqa: E731
    rho = col(0.5) * torch.exp(noise(0.01))
    b0 = math.sqrt(2.0 * math.exp(-2.0) / 100.0)
    return [rho, col(0.5) * noise(0.05), col(0.5) * noise(0.05), col(0.0) * noise(0.05),
            1.5 * rho * torch.exp(noise(0.01)), noise(0.1 * b0), noise(0.1 * b0), b0 + noise(0.1 * b0)]


def _fields(case, seed):
    """Per box the 8 fields [z, y, x], rounded to the case's type."""
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    make = {"orszag": _orszag, "turbulent": _turbulent, "stratified": _stratified}[case["state"]]
    dtype = getattr(torch, case["dtype"])
    return [[v.to(dtype).contiguous() for v in make(b, gen, dev)] for b in _boxes(case)]


def _weights(case, like, seed):
    """The cotangent of an adjoint step: order one, cell by cell."""
    gen = torch.Generator(device=like[0].device)
    gen.manual_seed(seed + 7919)
    return [torch.randn(t.shape, generator=gen, device=t.device, dtype=torch.float64).to(t.dtype) for t in like]


# ---------------------------------------------------------------------------
# one pass
def prepare(case, seed):
    from paper_2405_02483_amd import lib
    bits = lib.T_ALL
    for o in _options(case):
        bits |= getattr(lib, "T_" + o.upper())
    ctx = lib.Context(_boxes(case), dict(_params(case), terms=bits), dtype=getattr(torch, case["dtype"]))
    f = ctx.upload(_fields(case, seed))
    s = dict(case=case, ctx=ctx, f=f)
    kind = case["kind"]
    if case["tuned"]:
        ctx.autotune(f, reps=2)
    if kind == "step":
        s["work"] = (ctx.empty(), ctx.empty(), ctx.empty())
    elif kind in ("rhs", "monitor", "adjoint"):
        s["out"] = ctx.empty()
    if kind == "adjoint":
        s["g"] = _weights(case, f, seed)
    if kind == "rollout":
        s["f"] = [t.requires_grad_(True) for t in f]
    return s


def run(s):
    case, ctx, f = s["case"], s["ctx"], s["f"]
    kind = case["kind"]
    if kind == "step":          # dt = 0: each step's Courant dt, taken on the device
        return ctx.step(f, 0.0, case["steps"], work=s["work"])
    if kind == "rhs":
        return ctx.rhs(f, s["out"])
    if kind == "monitor":
        return {"dfdt": ctx.rhs(f, s["out"]), "stats": ctx.reductions(f, s["out"])}
    if kind == "clean":
        return ctx.divb_clean(f)[5:]
    if kind == "adjoint":
        return ctx.step_adjoint(f, _dt(case), s["g"], s["out"])
    from paper_2405_02483_amd.rollout import rollout
    y = rollout(ctx, f, _dt(case), case["steps"], ncheck=case["ncheck"])
    loss = sum((t * t).sum() for t in y)
    return {"y": [t.detach() for t in y], "grad": list(torch.autograd.grad(loss, f))}


def work(case):
    """Words: a step's three stages read and write the state and dU (24, 32
    and 24 per cell); a right-hand side 16; the reductions read state and dF;
    the projection reads and writes B; an adjoint step reads the state and a
    cotangent and writes one."""
    cells = sum(b["nx"] * b["ny"] * b["nz"] for b in _boxes(case))
    size, n = (8 if case["dtype"] == "float64" else 4), case["steps"]
    words, flops = {
        "step": (80 * n, 3 * RHS_FLOPS * n),
        "rhs": (16, RHS_FLOPS),
        "monitor": (32, RHS_FLOPS + 300),
        "clean": (6, 5 * 2 * math.log2(max(2, cells)) + 60),
        "adjoint": (24, 9 * RHS_FLOPS),
        "rollout": ((80 + 24) * n, (3 + 9) * RHS_FLOPS * n),
    }[case["kind"]]
    return {"bytes": float(words * cells * size), "flops": float(flops * cells)}


# ---------------------------------------------------------------------------
# the same in plain float64
DERIV = {1: (1.0,), 2: (9.0 / 8.0, -1.0 / 24.0), 3: (75.0 / 64.0, -25.0 / 384.0, 3.0 / 640.0)}
INTERP = {1: (0.5,), 2: (9.0 / 16.0, -1.0 / 16.0), 3: (75.0 / 128.0, -25.0 / 256.0, 3.0 / 256.0)}


def _spline_slopes(z):
    """dz/dk at the centres k and the faces k - 1/2 of the not-a-knot cubic
    spline through (k, z[k])."""
    n = len(z)
    z = torch.tensor(z, dtype=torch.float64)
    a, r = torch.zeros(n, n, dtype=torch.float64), torch.zeros(n, dtype=torch.float64)
    for row, at in ((0, 0), (n - 1, n - 3)):
        a[row, at:at + 3] = torch.tensor([1.0, -2.0, 1.0], dtype=torch.float64)
    for k in range(1, n - 1):
        a[k, k - 1:k + 2] = torch.tensor([1.0, 4.0, 1.0], dtype=torch.float64)
        r[k] = 6.0 * (z[k - 1] - 2.0 * z[k] + z[k + 1])
    m = torch.linalg.solve(a, r)

    def slope(k, t):
        return (z[k + 1] - z[k]) - (m[k + 1] - m[k]) / 6.0 + 0.5 * (m[k + 1] * t * t - m[k] * (1.0 - t) ** 2)
    return ([float(slope(min(k, n - 2), 0.0 if k < n - 1 else 1.0)) for k in range(n)],
            [float(slope(max(k, 1) - 1, 0.5 if k else -0.5)) for k in range(n)])


class Plain:
    """The staggered operators and the equations on one box."""

    def __init__(self, box, par, opts):
        self.b, self.p, self.opts = box, par, opts
        self.dev = _device()
        self.wall, self.n = box["wall"], box["nz"] + 2 * box["ngz"]
        self.h = (box["Lz"] / box["nz"], box["Ly"] / box["ny"], box["Lx"] / box["nx"])
        dzc = dzf = [self.h[0]] * self.n
        if box.get("zc"):
            dzc, dzf = _spline_slopes(box["zc"])
        self.dzc, self.dzf = self._col(dzc), self._col(dzf)
        self.hmin, self.hmax = min(self.h[1], self.h[2], min(dzc)), max(self.h[1], self.h[2], max(dzc))
        self.tables = {}

    def _col(self, v):
        return torch.tensor(v, device=self.dev, dtype=torch.float64).view(-1, 1, 1)

    def _table(self, der, up, top):
        """Coefficients [offset + 3][plane] of a z operator between walls: the
        widest centred stencil that fits, the unreachable end a copy."""
        key = (der, up, top)
        if key not in self.tables:
            n, t = self.n, [[0.0] * self.n for _ in range(7)]
            for k in range(n):
                c = k + up
                q = min(top, c, n - c)
                if q == 0:
                    c, q = (n - 1 if up else 1), 1
                # a stretched axis takes the Jacobian of the copied output
                jac = 1.0 / float((self.dzc if up else self.dzf)[c - up]) if der else 1.0
                for i, w in enumerate((DERIV if der else INTERP)[q]):
                    t[c + i - k + 3][k] += w * jac
                    t[c - 1 - i - k + 3][k] += (-w if der else w) * jac
            self.tables[key] = [self._col(v) for v in t]
        return self.tables[key]

    def op(self, f, ax, der, up, top=3):
        """Axes 0 z, 1 y, 2 x; up: to the index + 1/2 of the sample."""
        if ax == 0 and self.wall:
            g = torch.nn.functional.pad(f, (0, 0, 0, 0, 3, 3))
            return sum(t * g[d:d + self.n] for d, t in enumerate(self._table(der, up, top)))
        out = 0.0
        for i, w in enumerate((DERIV if der else INTERP)[top]):
            hi, lo = torch.roll(f, -(up + i), ax), torch.roll(f, -(up - 1 - i), ax)
            out = out + (w / self.h[ax] * (hi - lo) if der else w * (hi + lo))
        return out

    def dn(self, f, *axes):
        for a in axes:
            f = self.op(f, a, False, 0)
        return f

    def up(self, f, *axes):
        for a in axes:
            f = self.op(f, a, False, 1)
        return f

    def ddn(self, f, a, top=3):
        return self.op(f, a, True, 0, top)

    def dup(self, f, a, top=3):
        return self.op(f, a, True, 1, top)

    def beside(self, f, ax, fill):
        """f and its two neighbours along an axis (fill past a wall)."""
        if ax == 0 and self.wall:
            end = torch.full_like(f[:1], fill)
            return torch.cat([end, f[:-1]]), f, torch.cat([f[1:], end])
        return torch.roll(f, 1, ax), f, torch.roll(f, -1, ax)

    def max3(self, f, ax):
        return torch.stack(self.beside(f, ax, -math.inf)).max(dim=0).values

    def mean3(self, f, ax):
        n = 3.0
        if ax == 0 and self.wall:
            n = self._col([2.0] + [3.0] * (self.n - 2) + [2.0])
        return sum(self.beside(f, ax, 0.0)) / n

    def bend(self, f, ax):
        lo, mid, hi = self.beside(f, ax, 0.0)
        d = (lo - 2.0 * mid + hi).abs()
        if ax == 0 and self.wall:
            d = d * self._col([0.0] + [1.0] * (self.n - 2) + [0.0])
        return d

    @staticmethod
    def root(s):
        ok = s > 0
        return torch.where(ok, torch.where(ok, s, torch.ones_like(s)).sqrt(), torch.zeros_like(s))

    def speeds(self, f):
        """The smoothed viscosity with what the Courant condition reuses."""
        p, rho, e, B = self.p, f[0], f[4], f[5:]
        u = [m / self.dn(rho, 2 - a) for a, m in enumerate(f[1:4])]
        S = [self.dup(u[a], 2 - a) for a in range(3)]
        div = S[0] + S[1] + S[2]
        uc, bc = ([self.up(v[a], 2 - a) for a in range(3)] for v in (u, B))
        bb = self.root(bc[0] ** 2 + bc[1] ** 2 + bc[2] ** 2)
        wave = (p["gamma"] * (p["gamma"] - 1.0) * e / rho).sqrt() + bb / (p["mu"] * rho).sqrt()
        h = self.dzc.clamp(max=min(self.h[1], self.h[2])) if self.b.get("zc") else self.hmin
        nu = (p["nu1"] * self.root(uc[0] ** 2 + uc[1] ** 2 + uc[2] ** 2) + p["nu3"] * wave
              + p["nu2"] * h * torch.where(div < 0, -div, torch.zeros_like(div)))
        if "smag" in self.opts:
            off = [self.up(0.5 * (self.ddn(u[a], 2 - b) + self.ddn(u[b], 2 - a)), 2 - a, 2 - b)
                   for a, b in ((0, 1), (0, 2), (1, 2))]
            s2 = 2.0 * (sum(s * s for s in S) - div * div / 3.0 + 2.0 * sum(s * s for s in off))
            nu = nu + p["c_smag"] * h * self.root(s2)
        for a in (2, 1, 0):
            nu = self.max3(nu, a)
            if "max5" in self.opts:
                nu = self.max3(nu, a)
        for a in (2, 1, 0):
            nu = self.mean3(nu, a)
        return nu, u, S, div, uc, bc, bb, wave

    def courant(self, f):
        nu, _, _, _, uc, bc, bb, wave = self.speeds(self.fill(f))
        along = sum(a * b for a, b in zip(uc, bc)) / torch.where(bb > 0, bb, torch.ones_like(bb))
        perp = (sum(a * a for a in uc) - along * along).clamp(min=0.0).sqrt()
        inner = slice(self.b["ngz"], self.n - self.b["ngz"])
        diff = torch.maximum(nu, self.p["nuB"] * nu * (self.hmax / self.hmin))
        return min(self.p["Cdt"] * self.hmin / float((wave + perp)[inner].max()),
                   self.p["Cdtd"] * self.hmin / float(diff[inner].max()))

    def quench(self, t):
        s = sum(self.bend(t, a) for a in (2, 1, 0))
        den = t.abs() + s / self.p["q_max"]
        q = torch.where(den > 0, s / torch.where(den > 0, den, torch.ones_like(den)), torch.zeros_like(den))
        for a in (2, 1, 0):
            q = self.max3(q, a)
        return t * torch.where(q < self.p["q_lim"], q, torch.full_like(q, self.p["q_lim"]))

    def touching(self, m, *axes):
        for a in axes:
            m = m | self.beside(m, a, False)[0]
        return m

    def rate(self, f, dt=None):
        """The time derivatives on every plane, zero in the ghost planes."""
        p, o = self.p, self.opts
        rho, P3, e, B = f[0], f[1:4], f[4], f[5:]
        dn, up, ddn, dup = self.dn, self.up, self.ddn, self.dup
        X, Y, Z = 2, 1, 0
        ax = (X, Y, Z)
        nu, u, S, div = self.speeds(f)[:4]
        pr, em = (p["gamma"] - 1.0) * e, e / rho
        dx, dy = self.h[2], self.h[1]
        dzc, dzf = (self.dzc, self.dzf) if self.b.get("zc") else (self.h[0], self.h[0])
        longer = lambda a, b: b.clamp(min=a) if torch.is_tensor(b) else max(a, b)     # noqa: E731
        pairs = ((0, 1), (0, 2), (1, 2))
        length = (max(dx, dy), longer(dx, dzf), longer(dy, dzf))
        lnu = nu.log()
        edge = [length[q] * dn(lnu, ax[a], ax[b]).exp() for q, (a, b) in enumerate(pairs)]
        shear = [0.5 * (ddn(u[a], ax[b]) + ddn(u[b], ax[a])) for a, b in pairs]
        if "order2" in o:
            lr, lm = rho.log(), em.log()
            rough = torch.stack([self.bend(v, a) for v in (lr, lm) for a in ax]).amax(dim=0) > p["d2_lim"]
            S2 = [dup(u[a], ax[a], 1) for a in range(3)]
            S = [torch.where(rough, b, a) for a, b in zip(S, S2)]
            shear = [torch.where(self.touching(rough, ax[a], ax[b]),
                                 0.5 * (ddn(u[a], ax[b], 1) + ddn(u[b], ax[a], 1)), s)
                     for s, (a, b) in zip(shear, pairs)]
        tau = [rho * (l * nu) * s for l, s in zip((dx, dy, dzc), S)]
        tau_e = [dn(rho, ax[a], ax[b]) * edge[q] * shear[q] for q, (a, b) in enumerate(pairs)]
        if "quench" in o:
            tau, tau_e = [self.quench(t) for t in tau], [self.quench(t) for t in tau_e]
        # current, electric field (edge q = 0 xy holds the z component, ...)
        J = (ddn(B[2], Y) - ddn(B[1], Z), ddn(B[0], Z) - ddn(B[2], X), ddn(B[1], X) - ddn(B[0], Y))
        eta = [p["nuB"] * edge[q] for q in (2, 1, 0)]
        E = []
        for c in range(3):
            a, b = (c + 1) % 3, (c + 2) % 3
            E.append(eta[c] * J[c] - (dn(u[a], ax[b]) * dn(B[b], ax[a]) - dn(u[b], ax[a]) * dn(B[a], ax[b])))
        drho = -(dup(P3[0], X) + dup(P3[1], Y) + dup(P3[2], Z))
        if "lnp" in o:
            lpa = pr.mean(dim=(1, 2), keepdim=True).log().expand_as(pr)
            q = pr.log() - lpa
            grad = [(dn(lpa, a).exp() * dn(q, a).exp()) * (ddn(q, a) + ddn(lpa, a)) for a in ax]
        else:
            grad = [ddn(pr, a) for a in ax]
        which = {(0, 1): 0, (1, 0): 0, (0, 2): 1, (2, 0): 1, (1, 2): 2, (2, 1): 2}
        dp = []
        for a in range(3):
            d = ddn(tau[a] - up(P3[a], ax[a]) * up(u[a], ax[a]), ax[a]) - grad[a]
            for b in range(3):
                if b != a:
                    d = d + dup(tau_e[which[a, b]] - dn(P3[a], ax[b]) * dn(u[b], ax[a]), ax[b])
            b, c = (a + 1) % 3, (a + 2) % 3
            d = d + (up(J[b] * dn(B[c], ax[a]), ax[c]) - up(J[c] * dn(B[b], ax[a]), ax[b])) / p["mu"]
            dp.append(d)
        dp[2] = dp[2] - dn(rho, Z) * p["gz"]
        if "cori" in o:
            at = lambda v, a: dn(up(P3[v], ax[v]), ax[a])                             # noqa: E731
            w = p["omega"]
            for a in range(3):
                b, c = (a + 1) % 3, (a + 2) % 3
                dp[a] = dp[a] - 2.0 * (w[b] * at(c, a) - w[c] * at(b, a))
        de = -(pr * div) + sum(t * s for t, s in zip(tau, S))
        for q, (a, b) in enumerate(pairs):
            c = 3 - a - b
            de = de + up(2.0 * tau_e[q] * shear[q] + eta[c] * J[c] * J[c] / p["mu"], ax[a], ax[b])
        lne = em.log()
        for a, l in enumerate((dx, dy, dzf)):
            v = lne - em.mean(dim=(1, 2), keepdim=True).log() if a == 2 and "ediffav" in o else lne
            flux = p["nuE"] * dn(rho, ax[a]) * (l * dn(nu, ax[a])) * dn(em, ax[a]) * ddn(v, ax[a])
            de = de + dup(flux - dn(e, ax[a]) * u[a], ax[a])
        if "cool" in o:
            r2 = (rho / p["rho_cool"]) ** 2
            de = de - rho * (em - p["e_cool"]) / p["t_cool"] * (r2 / (1.0 + r2))
        dB = [dup(E[(c + 1) % 3], ax[(c + 2) % 3]) - dup(E[(c + 2) % 3], ax[(c + 1) % 3]) for c in range(3)]
        if "divb" in o and dt:
            db = sum(dup(B[a], ax[a]) for a in range(3))
            dB = [d + p["c_divb"] * self.hmin ** 2 / dt * ddn(db, ax[a]) for a, d in enumerate(dB)]
        out = [drho] + dp + [de] + dB
        if self.wall:
            g, k = self.b["ngz"], torch.arange(self.n, device=self.dev).view(-1, 1, 1)
            end = self.n - g
            for v in range(8):
                keep = (k >= g) & (k < end)
                if v == 3:
                    keep = (k > g) & (k < end)
                if v == 7:
                    keep = (k >= g) & (k <= end)
                out[v] = out[v] * keep
        return out

    def fill(self, f):
        """Ghost planes of closed walls: ln rho and ln e_m extrapolated, tangential
        velocities mirrored, tangential B and normal p antisymmetric."""
        if not self.wall:
            return list(f)
        g, n = self.b["ngz"], self.n
        end = n - g
        d = torch.arange(1, g + 1, device=self.dev, dtype=torch.float64).view(-1, 1, 1)

        def extended(v):
            v = v.log()
            lo = v[g] + d.flip(0) * (v[g] - v[g + 1])
            hi = v[end - 1] + d * (v[end - 1] - v[end - 2])
            return torch.cat([lo.exp(), v[g:end].exp(), hi.exp()])

        def keep(v, new):
            return torch.cat([new[:g], v[g:end], new[end:]])
        rho = keep(f[0], extended(f[0]))
        e = keep(f[4], rho * extended(f[4] / f[0]))

        def mirror(v, sign):
            return torch.cat([sign * v[g:2 * g].flip(0), v[g:end], sign * v[end - g:end].flip(0)])
        out = [rho, None, None, None, e, mirror(f[5], -1.0), mirror(f[6], -1.0), None]
        for a, ax in ((1, 2), (2, 1)):
            face = self.dn(rho, ax)
            out[a] = keep(f[a], face * mirror(f[a] / face, 1.0))

        def faces(v, sign, wall):
            lo, hi = v[g + 1:2 * g + 1].flip(0), v[end - g + 1:end].flip(0)
            first, last = (wall, wall) if wall is not None else (v[g:g + 1], v[end:end + 1])
            return torch.cat([sign * lo, first, v[g + 1:end], last, sign * hi])
        out[3], out[7] = faces(f[3], -1.0, torch.zeros_like(f[3][:1])), faces(f[7], 1.0, None)
        return out

    def step(self, f, dt):
        f, du = self.fill(f), None
        for s in range(3):
            F = self.rate(f, dt)
            du = F if du is None else [RK_ALPHA[s] * u + q for u, q in zip(du, F)]
            f = self.fill([v + RK_BETA[s] * dt * u for v, u in zip(f, du)])
        return f


def _solenoidal(P, f):
    """B minus the gradient of the potential of its discrete divergence."""
    div = P.dup(f[5], 2) + P.dup(f[6], 1) + P.dup(f[7], 0)
    k2 = 0.0
    for ax in range(3):
        n = div.shape[ax]
        th = torch.arange(n, device=div.device, dtype=torch.float64) * (2.0 * math.pi / n)
        k = sum(w * torch.sin((i + 0.5) * th) for i, w in enumerate(DERIV[3])) * (2.0 / P.h[ax])
        k2 = k2 + (k * k).view([n if a == ax else 1 for a in range(3)])
    k2[0, 0, 0] = 1.0
    ph = torch.fft.fftn(div) / -k2
    ph[0, 0, 0] = 0.0
    phi = torch.fft.ifftn(ph).real
    return [f[5] - P.ddn(phi, 2), f[6] - P.ddn(phi, 1), f[7] - P.ddn(phi, 0)]


def _totals(P, f):
    dv = P.h[1] * P.h[2] * P.dzc
    inner = slice(P.b["ngz"], P.n - P.b["ngz"])
    total = lambda v: float((v * dv)[inner].sum())                                    # noqa: E731
    none = ("divb_max", "divb_rms", "ratemax", "dt", "dt_wave", "dt_diff", "dt_rate", "dt_argmax", "dt_box",
            "dt_limit", "n_nonfinite", "n_nonpositive", "umax", "cmax", "numax", "mom", "bmax")
    return dict({k: None for k in none}, mass=total(f[0]), eint=total(f[4]),
                ekin=sum(total(0.5 * f[a] ** 2 / P.dn(f[0], 3 - a)) for a in (1, 2, 3)),
                emag=sum(total(v * v) for v in f[5:]) / (2.0 * P.p["mu"]))


def exact(case, seed):
    boxes, par, opts = _boxes(case), _params(case), _options(case)
    plain = [Plain(b, par, opts) for b in boxes]
    fields = [[v.double() for v in f] for f in _fields(case, seed)]
    kind = case["kind"]
    if kind == "step":
        for _ in range(case["steps"]):
            dt = min(P.courant(f) for P, f in zip(plain, fields))
            fields = [P.step(f, dt) for P, f in zip(plain, fields)]
        return [torch.cat([f[v].reshape(-1) for f in fields]) for v in range(8)]
    P, f = plain[0], fields[0]
    flat = lambda v: [t.detach().reshape(-1) for t in v]                              # noqa: E731
    if kind == "rhs":
        return flat(P.rate(P.fill(f)))
    if kind == "monitor":
        f = P.fill(f)
        return {"dfdt": flat(P.rate(f)), "stats": _totals(P, f)}
    if kind == "clean":
        return flat(_solenoidal(P, f))
    x = [v.requires_grad_(True) for v in f]
    y = x
    for _ in range(case["steps"]):
        y = P.step(y, _dt(case))
    if kind == "adjoint":
        like = [torch.empty(v.numel(), device=v.device, dtype=getattr(torch, case["dtype"])) for v in f]
        g = [w.double().view_as(v) for w, v in zip(_weights(case, like, seed), f)]
        return flat(torch.autograd.grad(y, x, grad_outputs=g))
    return {"y": flat(y), "grad": flat(torch.autograd.grad(sum((t * t).sum() for t in y), x))}

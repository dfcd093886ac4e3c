"""Timed cases of the FWIME operators, through the package's public entry points.

Each case is one call (or the pair of calls that always go together) of a
program that inverts for a velocity model: modeling of one shot, of a shot
set, with a free surface, and of a batch of uneven grids; the extended Born
pair, the objective with its gradients, the variable-projection step, the
autograd map, the time-lag pair, and the small vector work of the outer loop
(spline grid, L-BFGS direction).

Sizes are those of the repository's own workloads: the 100 x 200 problem with
11 offsets and nt = 1500, the request stream's grids (nz 200-600, nx 600-3000,
1-32 shots, 11 offsets), the batch's three grids, and the 300 x 1700
Marmousi-like set with 61 offsets or 101 lags of 16 ms, the last two with
fewer shots and a shorter record so that one call stays well below two seconds.
"""
import math

import numpy as np
import torch

import paper_2206_02362_amd as fwime

DEVICE = "cuda:0"
VMIN, VMAX = 1500.0, 4500.0
W = [-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0]
BATCH_GRIDS = ((200, 600), (300, 1700), (500, 2500))
EPS = 1e-3

_context = None


def context():
    """The one library context of the program (its scratch arena outlives the calls)."""
    global _context
    if _context is None:
        _context = fwime.Context(0)
    return _context


def listed():
    def grid(nz, nx, nb, nt, shots, nh=1, **more):
        return dict(nz=nz, nx=nx, nb=nb, nt=nt, shots=shots, nh=nh, dx=10.0, dt=8e-4, free_surface=False, **more)

    return [
        # the outer loop's model update: spline nodes -> grid, gradient -> nodes
        dict(name="spline_pair_300x1700", op="spline", nz=300, nx=1700, dx=10.0, step=10),
        # the outer loop's search direction over those nodes, 5 pairs
        dict(name="lbfgs_5x5985", op="lbfgs", n=5985, pairs=5),
        # one shot of a small model: nothing but launches
        dict(grid(100, 200, 40, 1500, 1), name="model_100x200_1shot", op="model"),
        # an ordinary modeling request: a few shots of one model
        dict(grid(300, 1400, 40, 1000, 8), name="model_300x1400_8shots", op="model"),
        # the free-surface-multiples variant, ragged grid, odd record
        dict(grid(217, 613, 40, 1501, 4), name="model_free_surface_217x613", op="model", free_surface=True),
        # many jobs of uneven grids in shared launches
        dict(name="batch_48_uneven", op="batch", jobs=48, nt=700, nb=40, dx=10.0, dt=8e-4),
        # the variable-projection step at a small size
        dict(grid(100, 200, 40, 1000, 2, 11, niter=3), name="vp_step_100x200_nh11", op="vp"),
        # extended modeling and migration of a shot set, wide offsets
        dict(grid(300, 1700, 60, 800, 8, 61), name="born_pair_300x1700_nh61", op="born"),
        # a training step through autograd at the small size
        dict(grid(100, 200, 40, 1500, 1, 11), name="autograd_100x200_nh11", op="autograd"),
        # an ordinary gradient request
        dict(grid(200, 600, 40, 1200, 4, 11), name="gradient_200x600_nh11", op="gradient"),
        # the full-width gradient, wide offsets
        dict(grid(300, 1700, 60, 800, 8, 61), name="gradient_300x1700_nh61", op="gradient"),
        # the time-lag pair, 101 lags of 16 ms
        dict(grid(300, 1700, 60, 1500, 2, 101, lag=20), name="tau_pair_300x1700_101lags", op="tau"),
    ]


def draw(rng):
    """A case of the same operators: depth 40-500, width 60-2500, strip 10-60, 1-16 shots, odd sizes among them."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["spline", "lbfgs", "model", "model", "model", "batch", "vp", "born", "born", "autograd",
                     "gradient", "gradient", "tau"])
    if op == "spline":
        return dict(op=op, nz=log(40, 500), nx=log(60, 2500), dx=10.0, step=rng.choice([6, 7, 8, 10]))
    if op == "lbfgs":
        return dict(op=op, n=log(500, 50000), pairs=rng.randint(1, 10))
    if op == "batch":
        return dict(op=op, jobs=log(3, 40), nt=rng.randint(200, 700), nb=rng.randint(20, 40), dx=10.0, dt=8e-4)
    top = max(work(c)["flops"] for c in listed() if c["op"] == op) if op not in ("autograd", "vp") else 2e11
    while True:
        c = dict(op=op, nz=log(40, 500), nx=log(60, 2500), nb=rng.randint(10, 60), nt=log(200, 2000),
                 shots=log(1, 16), nh=1, dx=rng.choice([7.5, 10.0, 12.5]), dt=8e-4,
                 free_surface=rng.random() < 0.2)
        if op != "model":
            c["nh"] = 2 * rng.randint(0, 30) + 1
        if op == "tau":
            c["lag"] = rng.randint(4, 24)
            c["nh"] = 2 * min(rng.randint(1, 50), 2 * c["nt"] // (2 * c["lag"])) + 1
            c["shots"] = min(c["shots"], 2)
        if op == "vp":
            c["niter"] = rng.randint(1, 3)
        if c["nh"] <= c["nx"] and work(c)["flops"] <= top:
            return c


# ---------------------------------------------------------------------------
# Inputs, made on the GPU from the seed
# ---------------------------------------------------------------------------
def _smooth(a, cells, axes):
    """Gaussian smoothing (periodic) of a device array along `axes`, scaled back to unit variance."""
    for ax in axes:
        k = torch.fft.rfftfreq(a.shape[ax], device=a.device)
        h = torch.exp(-2.0 * (math.pi * cells * k) ** 2)
        h = h.reshape([-1 if i == ax else 1 for i in range(a.dim())])
        a = torch.fft.irfft(torch.fft.rfft(a, dim=ax) * h, n=a.shape[ax], dim=ax)
    return a / a.std().clamp_min(1e-12)


def _randn(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEVICE)


def _velocity(gen, nx, nz, dx):
    """Smooth random medium (300 m correlation) between VMIN and VMAX."""
    a = _smooth(_randn(gen, nx, nz), 300.0 / dx, (0, 1))
    lo, hi = a.min(), a.max()
    return (VMIN + (a - lo) * ((VMAX - VMIN) / (hi - lo))).clamp(VMIN, VMAX).contiguous()


def _acquisition(gen, shots, nx, nt, dt):
    """Sources at random columns, a receiver on every column, both two cells deep; a Ricker wavelet of 6-12 Hz a shot."""
    src = torch.randint(0, nx, (shots,), generator=gen, device=DEVICE).cpu().numpy()
    f = 6.0 + 6.0 * torch.rand((shots, 1), generator=gen, device=DEVICE)
    a = (math.pi * f * (torch.arange(nt, device=DEVICE) * dt - 1.5 / f)) ** 2
    wav = ((1.0 - 2.0 * a) * torch.exp(-a)).contiguous()
    two = np.full(shots, 2)
    return fwime.Geometry(two, src, np.full((shots, nx), 2), np.tile(np.arange(nx), (shots, 1)), wav)


def _traces(gen, shots, nrec, nt, dt):
    """Band-limited traces (about 10 Hz at most) of order 1."""
    return _smooth(_randn(gen, shots, nrec, nt), 0.016 / dt, (2,)).contiguous()


def _nodes(n, d, step):
    """Spline nodes every `step` cells, twice as dense within two steps of a third of the axis."""
    at = np.arange(0, n - 1, step, dtype=np.float64)
    at = np.append(at, float(n - 1))
    mid = 0.5 * (at[1:] + at[:-1])
    return np.sort(np.concatenate([at, mid[np.abs(mid - n / 3.0) <= 2 * step]])) * d


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    op = case["op"]
    if op == "spline":
        zn, xn = _nodes(case["nz"], case["dx"], case["step"]), _nodes(case["nx"], case["dx"], case["step"])
        mc = 2500.0 + 500.0 * _smooth(_randn(gen, len(xn), len(zn)), 3.0, (0, 1))
        return dict(zn=zn, xn=xn, mc=mc.contiguous(), f=_smooth(_randn(gen, case["nx"], case["nz"]), 5.0, (0, 1)))
    if op == "lbfgs":
        s = _randn(gen, case["pairs"], case["n"])
        y = s * (0.5 + 1.5 * torch.rand((case["n"],), generator=gen, device=DEVICE))
        return dict(s=s, y=y, g=_randn(gen, case["n"]))
    if op == "batch":
        models = [_velocity(gen, nx, nz, case["dx"]) for nz, nx in BATCH_GRIDS]
        jobs = []
        for j in range(case["jobs"]):
            k = (j * 7 + j // 5) % 3
            nz, nx = BATCH_GRIDS[k]
            nt = case["nt"] - case["nt"] * ((j * 13) % 32) // 64       # between nt / 2 and nt
            grid = fwime.Grid(nz, nx, case["nb"], nt, case["dx"], case["dx"], case["dt"])
            jobs.append((grid, models[k], _acquisition(gen, 1, nx, nt, case["dt"])))
        return dict(jobs=jobs)
    nz, nx, nt, nh, shots, dx, dt = (case[k] for k in ("nz", "nx", "nt", "nh", "shots", "dx", "dt"))
    d = dict(grid=fwime.Grid(nz, nx, case["nb"], nt, dx, dx, dt, free_surface=case["free_surface"]),
             vel=_velocity(gen, nx, nz, dx), geom=_acquisition(gen, shots, nx, nt, dt))
    if op in ("born", "gradient", "autograd", "tau"):
        d["pt"] = (10.0 * _smooth(_randn(gen, nh, nx, nz), 2.0, (2,))).contiguous()
    if op in ("born", "tau"):
        d["data"] = _traces(gen, shots, nx, nt, dt)
    if op in ("gradient", "autograd", "vp"):                            # observed data, of the modeled data's order
        d["data"] = 1e-3 * _traces(gen, shots, nx, nt, dt)
    ih = np.arange(nh) - (nh - 1) // 2
    d["dso"] = np.sqrt(ih ** 2 + 1.0)
    return d


def prepare(case, seed):
    return dict(case=case, ctx=context(), **_inputs(case, seed))


def run(st):
    ctx, case = st["ctx"], st["case"]
    op = case["op"]
    if op == "spline":
        grid = (case["nz"], case["nx"], case["dx"], case["dx"], st["zn"], st["xn"])
        return ctx.spline_apply(*grid, st["mc"]), ctx.spline_adjoint(*grid, st["f"])
    if op == "lbfgs":
        return ctx.lbfgs_direction(st["s"], st["y"], st["g"])
    if op == "batch":
        return ctx.model_batch(st["jobs"])
    grid, vel, geom, nh = st["grid"], st["vel"], st["geom"], case["nh"]
    if op == "model":
        return ctx.model(grid, vel, geom)
    if op == "born":
        return ctx.born_ext_fwd(grid, vel, geom, st["pt"]), ctx.born_ext_adj(grid, vel, geom, st["data"], nh)
    if op == "tau":
        return (ctx.born_ext_tau_fwd(grid, vel, geom, st["pt"], case["lag"]),
                ctx.born_ext_tau_adj(grid, vel, geom, st["data"], nh, case["lag"]))
    if op == "gradient":
        return ctx.gradient(grid, vel, geom, st["pt"], st["data"], EPS, st["dso"])
    if op == "vp":
        return ctx.vp_solve(grid, vel, geom, st["data"], nh, EPS, st["dso"], case["niter"])
    v, p = st["vel"].clone().requires_grad_(True), st["pt"].clone().requires_grad_(True)
    pred = fwime.predicted_data(v, p, ctx, grid, geom)
    loss = 0.5 * (pred - st["data"]).square().sum()
    return (pred.detach(),) + torch.autograd.grad(loss, (v, p))


# ---------------------------------------------------------------------------
# What a pass cannot do without: inputs read and outputs written once, and the
# method's arithmetic (32 operations a cell update of the radius-4 stencil)
# ---------------------------------------------------------------------------
def work(case):
    op = case["op"]
    if op == "spline":
        n, m = case["nz"] * case["nx"], (case["nz"] // case["step"]) * (case["nx"] // case["step"])
        return {"bytes": 8.0 * n + 8.0 * m, "flops": 14.0 * n}
    if op == "lbfgs":
        return {"bytes": 4.0 * case["n"] * (2 * case["pairs"] + 2), "flops": 10.0 * case["n"] * case["pairs"]}
    if op == "batch":
        cells = sum((BATCH_GRIDS[(j * 7 + j // 5) % 3][0] + 2 * case["nb"])
                    * (BATCH_GRIDS[(j * 7 + j // 5) % 3][1] + 2 * case["nb"])
                    * (case["nt"] - case["nt"] * ((j * 13) % 32) // 64 - 1) for j in range(case["jobs"]))
        traces = sum(BATCH_GRIDS[(j * 7 + j // 5) % 3][1] for j in range(case["jobs"])) * case["nt"] * 0.75
        return {"bytes": 4.0 * traces + sum(4.0 * a * b for a, b in BATCH_GRIDS), "flops": 32.0 * cells}
    plane, steps = case["nz"] * case["nx"], case["shots"] * (case["nt"] - 1)
    padded = (case["nz"] + 2 * case["nb"]) * (case["nx"] + 2 * case["nb"])
    data, image = 4.0 * case["shots"] * case["nx"] * case["nt"], 4.0 * plane * case["nh"]
    cu, lag = 32.0 * padded * steps, 2.0 * plane * case["nh"] * steps
    prop, scat, arrays = {"model": (1, 0, data), "born": (4, 2, 2 * data + 2 * image),
                          "tau": (4, 2, 2 * data + 2 * image), "gradient": (4, 3, data + 2 * image),
                          "autograd": (4, 3, 2 * data + 2 * image),
                          "vp": (3 + 2 * case.get("niter", 1), 1 + 2 * case.get("niter", 1), data + image)}[op]
    return {"bytes": arrays + 4.0 * plane, "flops": prop * cu + scat * lag}


# ---------------------------------------------------------------------------
# The same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------
class _Medium:
    """Padded model of S shots: V = v^2 dt^2, the Cerjan taper, the offset geometry."""

    def __init__(self, grid, vel, geom):
        self.g, self.S, nb = grid, geom.nshots, grid.nb
        self.NX, self.NZ = grid.nx + 2 * nb, grid.nz + 2 * nb
        self.vel = vel.double()
        v = self.vel[(torch.arange(self.NX, device=DEVICE) - nb).clamp(0, grid.nx - 1)]
        v = v[:, (torch.arange(self.NZ, device=DEVICE) - nb).clamp(0, grid.nz - 1)]
        self.V = v ** 2 * grid.dt ** 2
        self.gam = self._taper(grid.nx)[:, None] * self._taper(grid.nz)[None, :]
        self.coef = 2.0 / (self.vel ** 3 * grid.dt ** 2)
        self.fs = nb if grid.free_surface else -1
        shots = torch.arange(self.S, device=DEVICE)
        at = [torch.as_tensor(a.astype(np.int64) + nb, device=DEVICE)
              for a in (geom.src_ix, geom.src_iz, geom.rec_ix, geom.rec_iz)]
        self.src, self.rec = (shots, at[0], at[1]), (shots[:, None], at[2], at[3])
        self.wav = geom.wavelet.double() / (grid.dx * grid.dz)

    def _taper(self, n):
        i = torch.arange(n + 2 * self.g.nb, device=DEVICE, dtype=torch.float64)
        k = (self.g.nb - i).clamp_min(0) + (i - (self.g.nb + n - 1)).clamp_min(0)
        return torch.exp(-(self.g.sponge_alpha * k / max(1, self.g.nb)) ** 2)

    def zeros(self):
        return torch.zeros((self.S, self.NX, self.NZ), device=DEVICE, dtype=torch.float64)

    def model_rows(self, a):
        return a[..., self.g.nb:self.g.nb + self.g.nz]

    def offsets(self, nh):
        """(h, model columns, source-side columns, receiver-side columns) whose columns lie on the padded grid."""
        nb, nx = self.g.nb, self.g.nx
        for ih in range(nh):
            h = ih - (nh - 1) // 2
            y0, y1 = max(0, abs(h) - nb), min(nx, self.NX - nb - abs(h))
            if y0 < y1:
                yield ih, slice(y0, y1), slice(nb + y0 - h, nb + y1 - h), slice(nb + y0 + h, nb + y1 + h)

    def source(self, n):
        return lambda r: r.index_put_(self.src, self.wav[:, n], accumulate=True)


class _Wave:
    """One field of the recursion; step() advances it and returns V (L u + source)."""

    def __init__(self, med):
        self.m = med
        shape = (med.S, med.NX + 8, med.NZ + 8)
        self.a, self.b = (torch.zeros(shape, device=DEVICE, dtype=torch.float64) for _ in range(2))

    @property
    def u(self):
        return self.a[:, 4:-4, 4:-4]

    def step(self, add=None):
        m, a, fs = self.m, self.a, self.m.fs
        if fs >= 0:
            for k in range(1, 5):
                a[:, :, 4 + fs - k] = -a[:, :, 4 + fs + k]
        idz, idx = 1.0 / m.g.dz ** 2, 1.0 / m.g.dx ** 2
        r = self.u * (W[0] * (idz + idx))
        nx, nz = m.NX, m.NZ
        for k in range(1, 5):
            r.add_(a[:, 4:4 + nx, 4 - k:4 - k + nz], alpha=W[k] * idz).add_(a[:, 4:4 + nx, 4 + k:4 + k + nz], alpha=W[k] * idz)
            r.add_(a[:, 4 - k:4 - k + nx, 4:4 + nz], alpha=W[k] * idx).add_(a[:, 4 + k:4 + k + nx, 4:4 + nz], alpha=W[k] * idx)
        if add is not None:
            add(r)
        r.mul_(m.V)
        if fs >= 0:
            r[:, :, :fs + 1] = 0.0
            a[:, :, :4 + fs] = 0.0
        old = self.b[:, 4:-4, 4:-4]
        old.mul_(m.gam).neg_().add_(self.u, alpha=2.0).add_(r).mul_(m.gam)
        if fs >= 0:
            old[:, :, :fs + 1] = 0.0
        self.a, self.b = self.b, self.a
        return r


def _scatter(m, c, t2, transpose=False):
    s = m.zeros()
    for ih, y, i, j in m.offsets(c.shape[0]):
        to, of = (i, j) if transpose else (j, i)
        m.model_rows(s)[:, to].addcmul_(m.model_rows(t2)[:, of], c[ih, y])
    return s


def _model(m, keep=False):
    nt = m.g.nt
    data = torch.zeros(tuple(m.rec[1].shape) + (nt,), device=DEVICE, dtype=torch.float64)
    hist, u = [], _Wave(m)
    for n in range(nt - 1):
        r = u.step(m.source(n))
        data[:, :, n + 1] = u.u[m.rec]
        if keep:
            hist.append(r)
    return data, hist


def _driven(m, sources, keep=False):
    """The field driven by dense sources: receiver data and V (L u + source) of every step."""
    data = torch.zeros(tuple(m.rec[1].shape) + (m.g.nt,), device=DEVICE, dtype=torch.float64)
    hist, w = [], _Wave(m)
    for n in range(m.g.nt - 1):
        r = w.step(lambda a, n=n: a.add_(sources(n)))
        data[:, :, n + 1] = w.u[m.rec]
        if keep:
            hist.append(r)
    return data, hist


def _adjoint(m, adj, each):
    """lambda_n for n = nt-2 .. 0, driven by `adj` at the receivers; each(n, lambda_n)."""
    lam = _Wave(m)
    for k in range(m.g.nt - 1, 0, -1):
        lam.step(lambda r: r.index_put_(m.rec, adj[:, :, k], accumulate=True))
        each(k - 1, lam.u)


def _image(m, hist, adj, nh):
    img = torch.zeros((nh, m.g.nx, m.g.nz), device=DEVICE, dtype=torch.float64)

    def each(n, lam):
        a, b = m.model_rows(hist[n]), m.model_rows(lam)
        for ih, y, i, j in m.offsets(nh):
            img[ih, y] += (a[:, i] * b[:, j]).sum(0)
    _adjoint(m, adj, each)
    return img * m.coef


def _gradient(m, hu, hd, adj, pt):
    """(grad_vel, B~^T adj)"""
    nh = pt.shape[0]
    c, gam = pt * m.coef, m.gam
    img, gp = torch.zeros_like(pt), torch.zeros((m.NX, m.NZ), device=DEVICE, dtype=torch.float64)
    rho, e = _Wave(m), [m.zeros(), m.zeros()]

    def each(n, lam):
        e.insert(0, _scatter(m, c, lam, True))
        rho.step(lambda r: r.add_(e[0] / gam - 2.0 * e[1] + gam * e[2]))
        e.pop()
        gp.add_(((hu[n] + hd[n]) * lam + hu[n] * rho.u).sum(0))
        a, b = m.model_rows(hu[n]), m.model_rows(lam)
        for ih, y, i, j in m.offsets(nh):
            img[ih, y] += (a[:, i] * b[:, j]).sum(0)
    _adjoint(m, adj, each)
    img *= m.coef
    nb, nx, nz = m.g.nb, m.g.nx, m.g.nz
    gx = gp[nb:nb + nx].clone()
    gx[0] += gp[:nb].sum(0)
    gx[-1] += gp[nb + nx:].sum(0)
    g = gx[:, nb:nb + nz].clone()
    g[:, 0] += gx[:, :nb].sum(1)
    g[:, -1] += gx[:, nb + nz:].sum(1)
    return g * m.coef - 3.0 / m.vel * (pt * img).sum(0), img


def _lagged(m, c, hist, lag):
    """Source of every step: sum_k c_k hist[n - 2 k lag] on the model grid."""
    K, ns, x = (c.shape[0] - 1) // 2, len(hist), slice(m.g.nb, m.g.nb + m.g.nx)

    def at(n):
        s = m.zeros()
        for k in range(-K, K + 1):
            if 0 <= n - 2 * k * lag < ns:
                m.model_rows(s)[:, x].addcmul_(m.model_rows(hist[n - 2 * k * lag])[:, x], c[k + K])
        return s
    return at


def _two_loop(s, y, g):
    q, k, rho, alpha = g.clone(), s.shape[0], [], []
    rho = [1.0 / torch.dot(s[i], y[i]) for i in range(k)]
    for i in reversed(range(k)):
        alpha.insert(0, rho[i] * torch.dot(s[i], q))
        q -= alpha[0] * y[i]
    q /= rho[-1] * torch.dot(y[-1], y[-1])
    for i in range(k):
        q += (alpha[i] - rho[i] * torch.dot(y[i], q)) * s[i]
    return -q


def _hat(nodes, n, d):
    """Dense [n][len(nodes)] matrix of the linear interpolation onto i d."""
    p = np.arange(n) * d
    c = np.clip(np.searchsorted(nodes, p, side="right") - 1, 0, len(nodes) - 2)
    t = np.clip((p - nodes[c]) / (nodes[c + 1] - nodes[c]), 0.0, 1.0)
    a = np.zeros((n, len(nodes)))
    a[np.arange(n), c] = 1.0 - t
    a[np.arange(n), c + 1] += t
    return torch.as_tensor(a, device=DEVICE)


def exact(case, seed):
    d, op = _inputs(case, seed), case["op"]
    if op == "spline":
        az, ax = _hat(d["zn"], case["nz"], case["dx"]), _hat(d["xn"], case["nx"], case["dx"])
        return ax @ d["mc"].double() @ az.T, ax.T @ d["f"].double() @ az
    if op == "lbfgs":
        return _two_loop(d["s"].double(), d["y"].double(), d["g"].double())
    if op == "batch":
        out = [None] * case["jobs"]
        for size in BATCH_GRIDS:                 # the jobs of one grid together, to the longest record
            mine = [j for j, (g, _, _) in enumerate(d["jobs"]) if (g.nz, g.nx) == size]
            if not mine:
                continue
            g, vel, _ = d["jobs"][mine[0]]
            nt = max(d["jobs"][j][0].nt for j in mine)
            geo = [d["jobs"][j][2] for j in mine]
            wav = torch.zeros((len(mine), nt), device=DEVICE)
            for i, a in enumerate(geo):
                wav[i, :a.wavelet.shape[1]] = a.wavelet[0]
            both = fwime.Geometry(*(np.concatenate([getattr(a, k) for a in geo])
                                    for k in ("src_iz", "src_ix", "rec_iz", "rec_ix")), wav)
            data, _ = _model(_Medium(fwime.Grid(g.nz, g.nx, g.nb, nt, g.dz, g.dx, g.dt), vel, both))
            for i, j in enumerate(mine):
                out[j] = data[i:i + 1, :, :d["jobs"][j][0].nt]
        return out
    m = _Medium(d["grid"], d["vel"], d["geom"])
    if op == "model":
        return _model(m)[0]
    f, hu = _model(m, keep=True)
    data, nh = d["data"].double(), case["nh"]
    if op == "vp":
        e2 = torch.as_tensor(EPS ** 2 * d["dso"] ** 2, device=DEVICE)[:, None, None]

        def normal(p):
            c = p * m.coef
            return _image(m, hu, _driven(m, lambda n: _scatter(m, c, hu[n]))[0], nh) + e2 * p
        res = data - f
        b = _image(m, hu, res, nh)
        p, r, s = torch.zeros_like(b), b.clone(), b.clone()
        phi = [0.5 * res.square().sum()]
        for _ in range(case["niter"]):
            q = normal(s)
            rr = r.square().sum()
            a = rr / (s * q).sum()
            p, r = p + a * s, r - a * q
            phi.append(phi[0] - 0.5 * ((b + r) * p).sum())
            s = r + (r.square().sum() / rr) * s
        return p, torch.stack(phi)
    pt = d["pt"].double()
    c = pt * m.coef
    if op == "tau":
        img, K, ns, x = torch.zeros_like(pt), (nh - 1) // 2, len(hu), slice(m.g.nb, m.g.nb + m.g.nx)

        def each(n, lam):
            for k in range(-K, K + 1):
                if 0 <= n - 2 * k * case["lag"] < ns:
                    img[k + K] += (m.model_rows(hu[n - 2 * k * case["lag"]])[:, x] * m.model_rows(lam)[:, x]).sum(0)
        _adjoint(m, data, each)
        return _driven(m, _lagged(m, c, hu, case["lag"]))[0], img * m.coef
    b, hd = _driven(m, lambda n: _scatter(m, c, hu[n]), keep=op != "born")
    if op == "born":
        return b, _image(m, hu, data, nh)
    r = f + b - data
    gv, gp = _gradient(m, hu, hd, r, pt)
    if op == "autograd":
        return f + b, gv, gp
    e2 = torch.as_tensor(EPS ** 2 * d["dso"] ** 2, device=DEVICE)[:, None, None]
    obj = 0.5 * r.square().sum() + 0.5 * (e2 * pt * pt).sum()
    return obj.reshape(1), gv, gp + e2 * pt

"""Workloads that a user of this framework runs, for timing them through the
public entry points of paper_2603_13618_amd.

Each listed case stands for a use:

* `shear128_f32`      a whole short run on a small D2Q9 grid, the double shear layer's 128^2: the
                      initial state and 100 steps in one call
* `step256_f32`       one step per call on a small grid: a loop that looks at the flags after each step
* `ragged_f32`        a D2Q9 grid whose sides are odd
* `smooth4096_f32`    the headline D2Q9 grid, FP32, row-interleaved state
* `smooth8192_bf16`   the largest grid, 16-bit population storage
* `ext2048_f32`       D2Q9 with every extension sensor it has
* `riemann2048_bgk`   D2Q25 finite volume, single distribution, four-quadrant Riemann problem
* `riemann1024_ddf`   D2Q25 double distribution (f, g), the grid of the paper's 2D Riemann runs
* `ragged_ddf_f64`    the double distribution in FP64 on a grid that is no multiple of a tile
* `sod1024_ddf`       the paper's shock tube, a pseudo-1D grid of two rows: the initial state and
                      64 steps in one call
* `adjoint1024_f32`   gradient of the summed KL sensor, forward and backward with checkpoints
* `cycle1024_f32`     one regridding cycle: steps, moments, macroscopic sensors, buffer layer, tile
                      counts, clustering on the host

`draw` gives more cases of the same kinds over the same ranges: grid sides from
48 to 8192 cells, all storage types, both layouts, any subset of the extension
sensors, periodic and outflow boundaries, 1 to 100 steps per call.
"""
import math

import numpy as np
import torch

from paper_2603_13618_amd import adjoint, lks

EXT9 = "kn,hr,sigma_h,sigma_hkl,alpha,shear,qh,comp,strain"
EXT25 = "kn,hr,sigma_h,sigma_hkl,alpha,shear,qh,qf"
EXTDDF = EXT25 + ",comp,strain"
GAMMA, PRANDTL = 1.4, 0.71
TAU = 0.52


def listed():
    return [
        dict(name="shear128_f32", kind="d2q9", field="shear", nx=128, ny=128, dtype="f32", layout="rows",
             steps=100, ext="", tau=0.55),
        dict(name="step256_f32", kind="d2q9", field="smooth", nx=256, ny=256, dtype="f32", layout="rows",
             steps=1, ext="", tau=TAU),
        dict(name="ragged_f32", kind="d2q9", field="smooth", nx=1023, ny=769, dtype="f32", layout="rows",
             steps=10, ext="", tau=TAU),
        dict(name="smooth4096_f32", kind="d2q9", field="smooth", nx=4096, ny=4096, dtype="f32",
             layout="rows", steps=10, ext="", tau=TAU),
        dict(name="smooth8192_bf16", kind="d2q9", field="smooth", nx=8192, ny=8192, dtype="bf16",
             layout="rows", steps=4, ext="", tau=TAU),
        dict(name="ext2048_f32", kind="d2q9", field="smooth", nx=2048, ny=2048, dtype="f32",
             layout="rows", steps=4, ext=EXT9, tau=TAU),
        dict(name="riemann2048_bgk", kind="d2q25", model="bgk", nx=2048, ny=2048, dtype="f32",
             layout="rows", steps=4, ext="", bc="outflow"),
        dict(name="riemann1024_ddf", kind="d2q25", model="ddf", nx=1024, ny=1024, dtype="f32",
             layout="rows", steps=4, ext="", bc="outflow"),
        dict(name="ragged_ddf_f64", kind="d2q25", model="ddf", nx=500, ny=301, dtype="f64",
             layout="rows", steps=4, ext="", bc="outflow"),
        dict(name="sod1024_ddf", kind="sod", model="ddf", nx=1024, ny=2, dtype="f32", layout="rows",
             steps=64, ext=""),
        dict(name="adjoint1024_f32", kind="adjoint", nx=1024, ny=1024, dtype="f32", layout="planes",
             steps=100, checkpoint=20, tau=TAU),
        dict(name="cycle1024_f32", kind="cycle", nx=1024, ny=1024, dtype="f32", layout="rows", steps=4,
             tau=TAU),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ranges.  Sides are log-uniform; half of them are
    rounded to a multiple of 64, the rest stay as drawn (odd ones among them)."""
    kind = rng.choice(["d2q9"] * 5 + ["d2q25"] * 4 + ["sod", "adjoint", "cycle"])
    layout = rng.choice(["rows", "rows", "planes"])

    def sides(lo, hi):
        nx, ny = _log_int(rng, lo, hi), _log_int(rng, lo, hi)
        if rng.random() < 0.5:
            nx, ny = max(64, nx // 64 * 64), max(64, ny // 64 * 64)
        return nx, ny

    if kind == "d2q9":
        dtype = rng.choice(["f32", "f32", "f32", "f64", "bf16", "f16"])
        nx, ny = sides(48, 6000)
        ext = ""
        if dtype in ("f32", "f64") and rng.random() < 0.25:
            names = EXT9.split(",")
            ext = ",".join(n for n in names if rng.random() < 0.5) or rng.choice(names)
        steps = min(_log_int(rng, 1, 100), max(1, 160_000_000 // (nx * ny)))
        return dict(kind="d2q9", field="smooth", nx=nx, ny=ny, dtype=dtype, layout=layout, steps=steps,
                    ext=ext, tau=round(rng.uniform(0.51, 0.8), 3))
    if kind == "d2q25":
        model = rng.choice(["bgk", "ddf"])
        dtype = rng.choice(["f32", "f32", "f32", "f64"])
        nx, ny = sides(48, 2048)
        ext = ""
        if rng.random() < 0.25:
            names = (EXTDDF if model == "ddf" else EXT25).split(",")
            ext = ",".join(n for n in names if rng.random() < 0.5) or rng.choice(names)
        cost = (2 if model == "ddf" else 1) * (3 if dtype == "f64" else 1) * (2 if ext else 1)
        # the first step starts from an equilibrium, whose sensors are rounding errors
        steps = max(2, min(_log_int(rng, 2, 50), 16_000_000 // (nx * ny * cost)))
        return dict(kind="d2q25", model=model, nx=nx, ny=ny, dtype=dtype, layout=layout, steps=steps,
                    ext=ext, bc=rng.choice(["outflow", "periodic"]))
    if kind == "sod":
        return dict(kind="sod", model=rng.choice(["bgk", "ddf"]), nx=_log_int(rng, 128, 2048), ny=2,
                    dtype=rng.choice(["f32", "f32", "f64"]), layout=layout, steps=rng.randint(8, 64), ext="")
    if kind == "adjoint":
        nx, ny = sides(48, 1024)
        steps = rng.randint(10, 100)
        return dict(kind="adjoint", nx=nx, ny=ny, dtype=rng.choice(["f32", "f32", "f64"]), layout=layout,
                    steps=steps, checkpoint=rng.randint(5, 25), tau=round(rng.uniform(0.51, 0.8), 3))
    nx, ny = sides(96, 1536)
    return dict(kind="cycle", nx=nx, ny=ny, dtype=rng.choice(["f32", "f32", "f64"]), layout=layout,
                steps=rng.randint(1, 8), tau=round(rng.uniform(0.51, 0.8), 3))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _device():
    return torch.device("cuda")


def _smooth_fields(nx, ny, seed):
    """rho, ux, uy: band-limited random Fourier series on a periodic grid."""
    dev = _device()
    gen = torch.Generator().manual_seed(int(seed))
    cut = max(1, min(16, nx // 12, ny // 12))
    k = torch.arange(-cut, cut + 1, dtype=torch.float64)

    def wave(n, ks):
        ph = 2.0 * math.pi * torch.outer(ks, torch.arange(n, dtype=torch.float64) / n)
        return torch.complex(torch.cos(ph), torch.sin(ph)).to(dev)

    ex, ey = wave(nx, k), wave(ny, k[cut:]).T
    out = []
    for _ in range(3):
        c = torch.randn(cut + 1, 2 * cut + 1, 2, generator=gen, dtype=torch.float64)
        c = torch.view_as_complex(c)
        c[0, : cut + 1] = 0
        norm = math.sqrt(2.0 * float(c.abs().square().sum()))
        out.append((2.0 / norm) * ((ey @ c.to(dev)) @ ex).real)
    return 1.0 + 0.01 * out[0], 0.03 * out[1], 0.03 * out[2]


def _shear_fields(nx, ny, seed):
    """The double shear layer, its perturbation's phase and size from the seed."""
    dev = _device()
    gen = torch.Generator().manual_seed(int(seed))
    a, b = (float(v) for v in torch.rand(2, generator=gen, dtype=torch.float64))
    x = (torch.arange(nx, dtype=torch.float64, device=dev) / nx)[None, :].expand(ny, nx)
    y = (torch.arange(ny, dtype=torch.float64, device=dev) / ny)[:, None].expand(ny, nx)
    ux = torch.where(y < 0.5, 0.05 * torch.tanh(80.0 * (y - 0.25)), 0.05 * torch.tanh(80.0 * (0.75 - y)))
    uy = 0.0025 * (0.5 + a) * torch.sin(2.0 * math.pi * (x + b))
    return torch.ones_like(ux), ux.contiguous(), uy.contiguous()


def _quadrant_fields(nx, ny, seed):
    """Four-quadrant Riemann problem with the states drawn from the seed."""
    dev = _device()
    gen = torch.Generator().manual_seed(int(seed))
    r = torch.rand(4, 4, generator=gen, dtype=torch.float64)
    rho, speed, ang, temp = 0.5 + r[:, 0], 0.1 * r[:, 1], 2.0 * math.pi * r[:, 2], 0.9 + 0.2 * r[:, 3]
    states = torch.stack([rho, speed * torch.cos(ang), speed * torch.sin(ang), temp]).to(dev)
    east = (torch.arange(nx, device=dev) >= nx // 2).long()[None, :]
    north = (torch.arange(ny, device=dev) >= ny // 2).long()[:, None]
    fields = states[:, 2 * north + east]
    smax = float((speed + torch.sqrt(2.0 * temp)).max())
    return [f.contiguous() for f in fields], smax


def _sod_fields(nx, ny, seed):
    """Sod's shock tube, the left state's pressure and the split moved a little by the seed."""
    dev = _device()
    gen = torch.Generator().manual_seed(int(seed))
    a, b = (float(v) for v in torch.rand(2, generator=gen, dtype=torch.float64))
    x = ((torch.arange(nx, dtype=torch.float64, device=dev) + 0.5) / nx)[None, :].expand(ny, nx)
    left = x <= 0.45 + 0.1 * a
    rho = torch.where(left, 1.0, 0.125).to(torch.float64).contiguous()
    p = torch.where(left, 0.95 + 0.1 * b, 0.1).to(torch.float64)
    zero = torch.zeros_like(rho)
    temp = (p / rho).contiguous()
    return [rho, zero, zero.clone(), temp], float(torch.sqrt(GAMMA * temp).max())


def _setup(case, seed):
    """Fields, constructor arguments and the plain numbers that exact() needs."""
    nx, ny = case["nx"], case["ny"]
    kw = dict(nx=nx, ny=ny, dtype=case["dtype"], layout=case["layout"], max_steps=max(1, case["steps"]))
    if case["kind"] in ("d2q9", "cycle", "adjoint"):
        fields = (_shear_fields if case.get("field") == "shear" else _smooth_fields)(nx, ny, seed)
        # near the 90th and 99th percentiles of a smooth field after a few steps on 4096^2,
        # scaled with its gradients
        g = 4096.0 * max(1.0 / nx, 1.0 / ny) * max(1, min(16, nx // 12, ny // 12)) / 16.0
        thr = [[4e-8 * g * g, 8e-8 * g * g], [2.2e-4 * g, 3.1e-4 * g], [1.3e-4 * g, 1.9e-4 * g],
               [math.inf, math.inf]]
        if case.get("field") == "shear":
            thr = [[7.6e-6, 1.3e-5], [1.4e-3, 1.9e-3], [1.8e-3, 2.4e-3], [math.inf, math.inf]]
        kw.update(lattice=9, tau=case["tau"], thr=thr, flag_mask=7)
        if case.get("ext"):
            kw["ext"] = case["ext"].split(",")
        return list(fields), kw
    ddf = case["model"] == "ddf"
    dx = 1.0 / max(nx, ny)
    if case["kind"] == "sod":
        fields, smax = _sod_fields(nx, ny, seed)
        mu, bc = 5e-4, (lks.OUTFLOW, lks.PERIODIC)
    else:
        fields, smax = _quadrant_fields(nx, ny, seed)
        mu = 1e-3
        bc = (lks.OUTFLOW, lks.OUTFLOW) if case["bc"] == "outflow" else (lks.PERIODIC, lks.PERIODIC)
    thr = [[4e-5, 4e-4], [6.8e-4, 6.8e-3], [1e-3, 1e-2], [5.8e-4, 5.8e-3]]
    kw.update(lattice=25, mu=mu, dt=0.01 * dx / smax, dx=dx, bc=bc, thr=thr, flag_mask=15)
    if ddf:
        kw.update(model="ddf", gamma=GAMMA, prandtl=PRANDTL, flag_mask=31, thr_qe=(6e-4, 6e-3))
    if case["ext"]:
        kw["ext"] = case["ext"].split(",")
    return fields, kw


def prepare(case, seed):
    fields, kw = _setup(case, seed)
    if case["kind"] == "adjoint":
        rho, ux, uy = fields
        return dict(case=case, rho=rho, ux=ux.requires_grad_(True), uy=uy.requires_grad_(True))
    lat = lks.Lattice(**kw)
    lat.init(*fields)
    return dict(case=case, lat=lat, fields=fields)


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] == "adjoint":
        loss = adjoint.kl_sensor_loss(state["ux"], state["uy"], state["rho"], tau=case["tau"],
                                      nsteps=case["steps"], checkpoint=case["checkpoint"],
                                      dtype=case["dtype"], layout=case["layout"])
        gux, guy = torch.autograd.grad(loss, (state["ux"], state["uy"]))
        return dict(loss=loss.detach(), gux=gux, guy=guy)
    lat = state["lat"]
    if case["kind"] == "sod" or case.get("field") == "shear":
        lat.init(*state["fields"])              # a whole short run, from its initial fields
    lat.step(case["steps"])
    out = dict(state=lat.state, sensors=lat.sensors, flags=lat.flags, sums=lat.sums)
    if case["kind"] == "cycle":
        rho, ux, uy, T = lat.moments()
        mac = lat.macro_sensors(rho, ux, uy, T, mu=case["tau"] / 3.0, per_rho=True,
                                which=("tau", "c", "s", "e", "qh"))
        levels = lat.tag_buffer(2)
        counts = lat.tag_tiles(levels, 1, 8)
        tiles = counts.cpu().numpy()
        boxes = lks.cluster(tiles, lat.nx, lat.ny, 8, eff=0.9, min_tiles=2)
        patches = np.full((tiles.size, 4), -1, np.int64)      # room for a patch per tile
        patches[: len(boxes)] = np.array(boxes, np.int64).reshape(-1, 4)
        out.update(moments=[rho, ux, uy, T], macro=[mac[n] for n in ("tau", "c", "s", "e", "qh")],
                   levels=levels, counts=counts, boxes=patches)
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    n, steps = case["nx"] * case["ny"], case["steps"]
    sb = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2}[case["dtype"]]
    rb = 8 if case["dtype"] == "f64" else 4
    if case["kind"] == "adjoint":
        # fields in, gradients out, the checkpoints written and read once; forward,
        # recomputed and reverse steps at about 120, 120 and 250 operations a cell
        kept = -(-steps // case["checkpoint"])
        return dict(bytes=n * (24 + 16 + 2 * 9 * sb * kept), flops=n * steps * 490)
    if case["kind"] in ("d2q9", "cycle"):
        next_ = len(case["ext"].split(",")) if case.get("ext") else 0
        b = n * (2 * 9 * sb + (3 + next_) * rb + 1) + 64 * steps
        f = n * steps * (250 + 60 * next_)
        if case["kind"] == "cycle":
            b += n * (4 * 8 + 5 * 8 + 1)
            f += n * 160
        return dict(bytes=b, flops=f)
    ddf = case["model"] == "ddf"
    q, planes = (50, 5) if ddf else (25, 4)
    next_ = len(case["ext"].split(",")) if case["ext"] else 0
    return dict(bytes=n * (2 * q * sb + (planes + next_) * rb + 1) + 64 * steps,
                flops=n * steps * (q * 75 + 25 * 8 * next_))


# --------------------------------------------------------------------------
# the same in 64 bits, plain torch
# --------------------------------------------------------------------------
_GH3 = ([-1.0, 0.0, 1.0], [1.0 / 6.0, 2.0 / 3.0, 1.0 / 6.0])


def _cells(v):
    return torch.tensor(v, dtype=torch.float64, device=_device())[:, None, None]


def _log_ratio_sum(f, feq):
    return (f * torch.log(f / feq)).sum(0)


class _D2Q9:
    def __init__(self, tau):
        x, w = _GH3
        self.c = [(int(x[i // 3]), int(x[i % 3])) for i in range(9)]
        self.w = _cells([w[i // 3] * w[i % 3] for i in range(9)])
        self.cx, self.cy = _cells([c[0] for c in self.c]), _cells([c[1] for c in self.c])
        self.tau = tau

    def equilibrium(self, rho, ux, uy):
        cu = self.cx * ux + self.cy * uy
        return self.w * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * (ux * ux + uy * uy))

    def pull(self, f):
        return torch.stack([torch.roll(f[i], (cy, cx), (0, 1)) for i, (cx, cy) in enumerate(self.c)])

    def moments(self, f):
        rho = f.sum(0)
        return rho, (self.cx * f).sum(0) / rho, (self.cy * f).sum(0) / rho

    def collide(self, g):
        rho, ux, uy = self.moments(g)
        feq = self.equilibrium(rho, ux, uy)
        return g - (g - feq) / self.tau, feq, rho, ux, uy

    def kl(self, g, feq):
        return (g * torch.log(g / feq) - g + feq).sum(0)


def _extension(names, f, feq, w, P, u, mu, omega, q=None, bulk=None):
    """The extension sensors of one or two distributions (lists of f, f^eq, w, Omega)."""
    pxx, pxy, pyy = P
    out = {}
    fneq = [a - b for a, b in zip(f, feq)]
    if "kn" in names:
        out["kn"] = sum((n / e).abs().sum(0) for n, e in zip(fneq, feq))
    if "hr" in names:
        out["hr"] = sum(((a * torch.log(a / v)).sum(0) - (e * torch.log(e / v)).sum(0)).abs()
                        for a, e, v in zip(f, feq, w))
    if "sigma_h" in names:
        out["sigma_h"] = -sum((o * torch.log(a / v)).sum(0) for o, a, v in zip(omega, f, w))
    if "sigma_hkl" in names:
        out["sigma_hkl"] = -sum((o * torch.log(a / e)).sum(0) for o, a, e in zip(omega, f, feq))
    if "alpha" in names:
        tot = 0.0
        for n, a in zip(fneq, f):
            m = [((-1.0) ** (k - 1) / (k * (k + 1)) * n ** (k + 1) / a ** k).sum(0) for k in range(1, 5)]
            r2, r3, r4 = m[1] / m[0], m[2] / m[0], m[3] / m[0]
            d = 4 * r2 - 16 * r2 ** 2 + 8 * r3 - 80 * r2 * r3 + 80 * r2 ** 3 + 16 * r4
            tot = tot + torch.where(m[0] != 0, d, torch.zeros_like(d)).abs()
        out["alpha"] = tot
    hx, hy = u[0] * pxx + u[1] * pxy, u[0] * pxy + u[1] * pyy
    if "shear" in names:
        out["shear"] = torch.sqrt(0.5 * (pxx - pyy) ** 2 + 2 * pxy ** 2) / mu
    if "qh" in names:
        out["qh"] = torch.sqrt(hx ** 2 + hy ** 2)
    if "qf" in names:
        out["qf"] = torch.sqrt((q[0] - hx) ** 2 + (q[1] - hy) ** 2)
    if "comp" in names:
        out["comp"] = math.sqrt(2.0) * (pxx + pyy).abs() / (2 * mu * bulk[0])
    if "strain" in names:
        t = bulk[1] * (pxx + pyy)
        out["strain"] = torch.sqrt((t - pxx) ** 2 + 2 * pxy ** 2 + (t - pyy) ** 2) / (2 * mu)
    return [out[n] for n in lks.EXT_NAMES if n in names]


def _exact_d2q9(case, fields):
    rho, ux, uy = fields
    m = _D2Q9(case["tau"])
    f = m.equilibrium(rho, ux, uy)
    sums = []
    for s in range(case["steps"]):
        g = m.pull(f)
        f, feq, r, u, v = m.collide(g)
        neq = g - feq
        pxx, pxy, pyy = (m.cx * m.cx * neq).sum(0), (m.cx * m.cy * neq).sum(0), (m.cy * m.cy * neq).sum(0)
        sens = [m.kl(g, feq), neq.abs().sum(0), torch.sqrt(pxx ** 2 + 2 * pxy ** 2 + pyy ** 2)]
        zero = torch.zeros((), dtype=torch.float64, device=f.device)
        sums.append(torch.stack([r.sum(), (r * u).sum(), (r * v).sum(), zero] + [p.sum() for p in sens] + [zero]))
    if case.get("ext"):
        mu = case["tau"] * r / 3.0
        # lambda = 0: 2 mu + D lambda = 2 mu; no trace term in the strain
        sens += _extension(case["ext"].split(","), [g], [feq], [m.w], (pxx, pxy, pyy), (u, v), mu,
                           [-neq / case["tau"]], bulk=(1.0, 0.0))
    return m, f, torch.stack(sens), torch.stack(sums)


class _D2Q25:
    def __init__(self, model):
        x, w = np.polynomial.hermite_e.hermegauss(5)
        w = w / w.sum()
        self.x, self.w1 = [float(v) for v in x], [float(v) for v in w]
        self.w = _cells([w[i // 5] * w[i % 5] for i in range(25)])
        self.vx, self.vy = _cells([x[i // 5] for i in range(25)]), _cells([x[i % 5] for i in range(25)])
        self.v2 = self.vx ** 2 + self.vy ** 2
        self.model = model

    @staticmethod
    def _he(x):
        return [1.0, x, (x * x - 1.0) / 2.0, (x ** 3 - 3.0 * x) / 6.0, (x ** 4 - 6.0 * x * x + 3.0) / 24.0]

    @staticmethod
    def _h(u, t):
        return [torch.ones_like(u), u, u * u + t, u ** 3 + 3 * u * t, u ** 4 + 6 * u * u * t + 3 * t * t]

    def equilibrium(self, rho, ux, uy, T):
        hx, hy = self._h(ux, T - 1.0), self._h(uy, T - 1.0)
        out = torch.empty((25,) + tuple(rho.shape), dtype=torch.float64, device=rho.device)
        for a in range(5):
            ea = self._he(self.x[a])
            px = [ea[n] * hx[n] for n in range(5)]
            for b in range(5):
                eb = self._he(self.x[b])
                s = 0.0
                for k in range(5):
                    s = s + px[k] * sum(eb[n] * hy[n] for n in range(5 - k))
                out[5 * a + b] = self.w1[a] * self.w1[b] * rho * s
        return out

    def _pad(self, f, bc, dim):
        n = f.shape[dim]
        idx = torch.arange(-2, n + 2, device=f.device)
        idx = idx.clamp(0, n - 1) if bc == lks.OUTFLOW else idx % n
        return f.index_select(dim, idx)

    def _div(self, f, v, bc, dim):
        """v dF/dx of one population: upwind, van Leer limited; f [ny, nx], v a number."""
        n = f.shape[dim]
        p = self._pad(f, bc, dim)
        d = p.narrow(dim, 1, n + 3) - p.narrow(dim, 0, n + 3)
        a, b = d.narrow(dim, 0, n + 2), d.narrow(dim, 1, n + 2)
        ab = a * b
        h = torch.where(ab > 0, ab / torch.where(ab > 0, a + b, torch.ones_like(a)), torch.zeros_like(a))
        c = p.narrow(dim, 1, n + 2)                       # cells -1 .. n with their half slopes h
        face = (c + h).narrow(dim, 0, n + 1) if v > 0 else (c - h).narrow(dim, 1, n + 1)
        return v * (face.narrow(dim, 1, n) - face.narrow(dim, 0, n))

    def advect(self, f, bc):
        """sum over both directions, bc = (bc_x, bc_y)."""
        out = torch.zeros_like(f)
        for i in range(25):
            a, b = self.x[i // 5], self.x[i % 5]
            if i // 5 != 2:
                out[i] += self._div(f[i], a, bc[0], 1)
            if i % 5 != 2:
                out[i] += self._div(f[i], b, bc[1], 0)
        return out


def _exact_d2q25(case, fields, kw):
    m = _D2Q25(case["model"])
    ddf = case["model"] == "ddf"
    rho, ux, uy, T = fields
    mu, dt, dx, bc = kw["mu"], kw["dt"], kw["dx"], kw["bc"]
    cv = 1.0 / (GAMMA - 1.0)
    f = m.equilibrium(rho, ux, uy, T)
    g = (cv - 1.0) * T * f if ddf else None
    sums = []
    for s in range(case["steps"]):
        r = f.sum(0)
        u, v = (m.vx * f).sum(0) / r, (m.vy * f).sum(0) / r
        e = 0.5 * (m.v2 * f).sum(0)
        if ddf:
            e = e + g.sum(0)
            T = (e / r - 0.5 * (u * u + v * v)) / cv
        else:
            T = e / r - 0.5 * (u * u + v * v)
        feq = m.equilibrium(r, u, v, T)
        neq = f - feq
        it1 = r * T / mu
        pxx, pxy, pyy = (m.vx ** 2 * neq).sum(0), (m.vx * m.vy * neq).sum(0), (m.vy ** 2 * neq).sum(0)
        qx, qy = (0.5 * m.v2 * m.vx * neq).sum(0), (0.5 * m.v2 * m.vy * neq).sum(0)
        kl = _log_ratio_sum(f, feq)
        bad = ((f <= 0) | (feq <= 0)).any(0)
        sneq = neq.abs().sum(0)
        om_f = -it1 * neq
        if ddf:
            geq = (cv - 1.0) * T * feq
            gneq = g - geq
            c2 = (m.vx - u) ** 2 + (m.vy - v) ** 2
            qf = [(0.5 * c2 * (c - w_) * neq).sum(0) for c, w_ in ((m.vx, u), (m.vy, v))]
            qg = [((c - w_) * gneq).sum(0) for c, w_ in ((m.vx, u), (m.vy, v))]
            fs = m.w * (qf[0] * m.vx + qf[1] * m.vy) * (0.25 * m.v2 - 1.0)
            gs = m.w * (qg[0] * m.vx + qg[1] * m.vy)
            it12 = it1 * (1.0 - PRANDTL)
            om_f = om_f + it12 * fs
            om_g = -it1 * gneq + it12 * gs
            qx, qy = qx + (m.vx * gneq).sum(0), qy + (m.vy * gneq).sum(0)
            kl = kl.abs() + _log_ratio_sum(g, geq).abs()
            bad = bad | ((g <= 0) | (geq <= 0)).any(0)
            sneq = sneq + gneq.abs().sum(0)
        kl = torch.where(bad, torch.full_like(kl, math.inf), kl)
        sens = [kl, sneq, torch.sqrt(pxx ** 2 + 2 * pxy ** 2 + pyy ** 2), torch.sqrt(qx ** 2 + qy ** 2)]
        sums.append(torch.stack([r.sum(), (r * u).sum(), (r * v).sum(), e.sum()] + [p.sum() for p in sens]))
        if ddf:
            sens.append(fs.abs().sum(0) + gs.abs().sum(0))
        if s + 1 == case["steps"] and case["ext"]:
            bulk = (1.0 - 1.0 / cv, -1.0 / (2.0 * (cv - 1.0))) if ddf else None
            sens += _extension(case["ext"].split(","), [f] + ([g] if ddf else []), [feq] + ([geq] if ddf else []),
                               [m.w] + ([m.w] if ddf else []), (pxx, pxy, pyy), (u, v), mu,
                               [om_f] + ([om_g] if ddf else []), q=(qx, qy), bulk=bulk)
        f = f - dt / dx * m.advect(f, bc) + dt * om_f
        if ddf:
            g = g - dt / dx * m.advect(g, bc) + dt * om_g
    dev = f - m.w
    if ddf:
        dev = torch.cat([dev, g - (cv - 1.0) * m.w])
    return dev, torch.stack(sens), torch.stack(sums)


def _exact_adjoint(case, fields):
    rho, ux, uy = fields
    m = _D2Q9(case["tau"])
    states = [m.equilibrium(rho, ux, uy)]
    for _ in range(case["steps"] - 1):
        states.append(m.collide(m.pull(states[-1]))[0])
    lam = None
    loss = None
    for n in range(case["steps"], 0, -1):
        f = states.pop().requires_grad_(True)
        g = m.pull(f)
        out, feq = m.collide(g)[:2]
        if lam is None:
            loss = m.kl(g, feq).sum()
            lam, = torch.autograd.grad(loss, f)
        else:
            lam, = torch.autograd.grad(out, f, lam)
    u, v = ux.clone().requires_grad_(True), uy.clone().requires_grad_(True)
    gux, guy = torch.autograd.grad(m.equilibrium(rho, u, v), (u, v), lam)
    return dict(loss=loss.detach(), gux=gux, guy=guy)


def _exact_macro(case, rho, ux, uy):
    def dd(a, dim):
        return 0.5 * (torch.roll(a, -1, dim) - torch.roll(a, 1, dim))

    mu = case["tau"] / 3.0 * rho
    xx, yy, xy = dd(ux, 1), dd(uy, 0), dd(uy, 1) + dd(ux, 0)
    div = xx + yy
    txx, tyy, txy = -2 * mu * xx, -2 * mu * yy, -mu * xy
    return [torch.sqrt(txx ** 2 + tyy ** 2 + 2 * txy ** 2), math.sqrt(2.0) * div.abs(),
            torch.sqrt((2 * xx - div) ** 2 + (2 * yy - div) ** 2 + 2 * xy ** 2),
            torch.sqrt(xx ** 2 + yy ** 2 + 0.5 * xy ** 2),
            torch.sqrt((ux * txx + uy * txy) ** 2 + (ux * txy + uy * tyy) ** 2)]


def exact(case, seed):
    cells = case["nx"] * case["ny"]
    if case["kind"] in ("d2q25", "sod") and cells * case["steps"] > 40_000_000:
        return None
    fields, kw = _setup(case, seed)
    half = case["dtype"] in ("bf16", "f16")
    if case["kind"] == "adjoint":
        return _exact_adjoint(case, fields)
    if case["kind"] in ("d2q25", "sod"):
        dev, sens, sums = _exact_d2q25(case, fields, kw)
        # alpha is a ratio of rounding errors in the quadrants that are still uniform
        alpha = "alpha" in case["ext"].split(",")
        return dict(state=dev, sensors=None if alpha else sens, flags=None, sums=sums)
    m, f, sens, sums = _exact_d2q9(case, fields)
    # 16-bit storage rounds the non-equilibrium parts themselves: the sensors
    # have no 64-bit value to be compared with
    out = dict(state=f - m.w, sensors=None if half else sens, flags=None, sums=None if half else sums)
    if case["kind"] == "cycle":
        rho, ux, uy = m.moments(f)
        out.update(moments=[rho, ux, uy, torch.full_like(rho, 1.0 / 3.0)], macro=_exact_macro(case, rho, ux, uy),
                   levels=None, counts=None, boxes=None)
    return out

"""The work that users of this library have it do, as measurable cases.

Every case is a dict of plain values; `prepare` makes what a user's program holds before the call
(inputs from the seed, kernel sets, plans, networks), `run` is one pass through the public entry
points, `work` is what the pass cannot do without and `exact` the same outputs in 64 bits, written
here from the definitions with torch alone.

Sky and array are those of the library's own workloads: 36 antennas in a disk tracked over eight
hours, a Gaussian power beam of one degree with 1 % leakage, w-planes spaced evenly, supports from
16 to 48 taps by the library's support rule, eight-fold oversampling.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2206_15117_amd import autotune, clean
from paper_2206_15117_amd import polgrid as pg

DEG = math.pi / 180.0
C_LIGHT = 299792458.0
LAT, DEC = -26.7 * DEG, -45.0 * DEG
N_ANT, N_BASE = 36, 630
AA = 7  # support of the anti-aliasing function


# ---------------------------------------------------------------------------------------- the cases

def listed():
    return [
        # one Stokes-I snapshot, everything included: the smallest call, bound by latency
        dict(name="stokes_i_step", kind="stokes_step", n=256, rows=20000, planes=8, support=7, os=4, fov=0.1),
        # a short full-polarisation observation imaged once from new data: plan, image, residual
        dict(name="snapshot_cycle", kind="cycle", n=1024, rows=62370, planes=16, fov=0.06, mhz=1400.0, chans=1, keep_plan=False),
        # the stages of an eight-hour full-polarisation track, one by one: binning, ...
        dict(name="fullpol_plan", kind="plan", n=2048, rows=2300000, planes=32, fov=0.0695, mhz=1400.0, chans=1),
        # ... gridding onto 2048^2 x 4 through float32 kernel tables, ...
        dict(name="fullpol_grid", kind="grid", n=2048, rows=2300000, planes=32, fov=0.0695, mhz=1400.0, chans=1, storage=0, exactly=False),
        # ... and degridding a model from the same grid
        dict(name="fullpol_degrid", kind="degrid", n=2048, rows=2300000, planes=32, fov=0.0695, mhz=1400.0, chans=1, storage=0),
        # gridding with the same bits on every call, on a ragged row count
        dict(name="reproducible_grid", kind="grid", n=1500, rows=701317, planes=24, fov=0.06, mhz=1100.0, chans=1, storage=0, exactly=True),
        # several channels, each with its own kernels, grid and row count, in one launch each way; float16 tables
        dict(name="channel_batch", kind="batch", n=2048, rows_lo=100000, rows_hi=1500000, fields=5, planes=32, fov=0.0695),
        # one major cycle of a many-channel observation with its plan kept: image, predict, subtract
        dict(name="major_cycle", kind="cycle", n=4096, rows=6000000, planes=64, fov=0.07, mhz=1295.5, chans=96, keep_plan=True),
        # kernel tables for one pointing from its Jones field, gridding direction
        dict(name="kernel_set", kind="kernels", n=2048, planes=24, fov=0.0695, mk=256, direction=0, storage=0),
        # the minor cycle of clean on a four-plane residual
        dict(name="clean_minor", kind="clean", n=1536, npol=4, iters=400, patch=200),
        # a field image put onto the mosaic frame with its weights, and the model brought back
        dict(name="mosaic_resample", kind="resample", n=3000, npol=4, pad=1.25, offset=0.5),
        # one training step of the kernel network in basis coordinates
        dict(name="network_train", kind="train", features=24, width=256, hidden=3, outputs=256, batch=1024),
    ]


def _log_int(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    kind = rng.choice(["stokes_step", "cycle", "plan", "grid", "grid", "degrid", "degrid", "batch", "cycle_kept",
                       "kernels", "clean", "resample", "train"])
    fov = round(rng.uniform(0.045, 0.072), 4)
    mhz = round(rng.uniform(700.0, 1800.0), 1)
    if kind == "stokes_step":
        return dict(kind=kind, n=2 * rng.randrange(64, 513), rows=_log_int(rng, 3000, 200000), planes=rng.randrange(3, 17),
                    support=rng.choice([6, 7, 8, 9, 11]), os=rng.choice([4, 8]), fov=round(rng.uniform(0.05, 0.1), 4))
    if kind == "cycle":
        return dict(kind="cycle", n=2 * rng.randrange(256, 1025), rows=_log_int(rng, 10000, 400000),
                    planes=rng.randrange(8, 33), fov=fov, mhz=mhz, chans=rng.choice([1, 1, 4]), keep_plan=False)
    if kind == "cycle_kept":
        return dict(kind="cycle", n=2 * rng.randrange(768, 2049), rows=_log_int(rng, 400000, 4000000),
                    planes=rng.randrange(24, 65), fov=fov, mhz=mhz, chans=rng.choice([4, 16, 96]), keep_plan=True)
    if kind == "plan":
        return dict(kind=kind, n=2 * rng.randrange(256, 2049), rows=_log_int(rng, 20000, 6000000),
                    planes=rng.randrange(8, 65), fov=fov, mhz=mhz, chans=rng.choice([1, 4, 16]))
    if kind in ("grid", "degrid"):
        c = dict(kind=kind, n=2 * rng.randrange(400, 1401), rows=_log_int(rng, 100000, 2500000),
                 planes=rng.randrange(12, 41), fov=fov, mhz=mhz, chans=rng.choice([1, 1, 8]), storage=rng.choice([0, 0, 0, 1]))
        if kind == "grid":
            c["exactly"] = rng.random() < 0.3
        return c
    if kind == "batch":
        lo = _log_int(rng, 50000, 200000)
        return dict(kind=kind, n=2 * rng.randrange(512, 1025), rows_lo=lo, rows_hi=lo * rng.randrange(3, 8),
                    fields=rng.randrange(2, 7), planes=rng.randrange(12, 33), fov=fov)
    if kind == "kernels":
        return dict(kind=kind, n=2 * rng.randrange(512, 1401), planes=rng.randrange(4, 29), fov=fov,
                    mk=rng.choice([128, 192, 256]), direction=rng.choice([0, 1]), storage=rng.choice([0, 0, 1]))
    if kind == "clean":
        return dict(kind=kind, n=2 * rng.randrange(256, 1025), npol=rng.choice([1, 4]), iters=_log_int(rng, 50, 500),
                    patch=_log_int(rng, 60, 400))
    if kind == "resample":
        return dict(kind=kind, n=2 * rng.randrange(512, 1601), npol=rng.choice([1, 4]), pad=round(rng.uniform(1.0, 1.4), 2),
                    offset=round(rng.uniform(0.1, 0.8), 2))
    return dict(kind="train", features=rng.randrange(12, 33), width=rng.choice([128, 256]), hidden=rng.choice([2, 3]),
                outputs=rng.choice([128, 200, 256]), batch=_log_int(rng, 128, 1024))


# ------------------------------------------------------------------------------- inputs from the seed

def _rng(seed, salt):
    return np.random.default_rng([int(seed), salt])


def _torch_gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _uvw(rows, n, fov, mhz, chans, seed, every=1):
    """Earth-rotation tracks of 36 antennas whose longest baseline spans the grid, channel-major and
    time-major rows, float64 [rows][3] in wavelengths; `every`: only each so many-th row."""
    rng = _rng(seed, 1)
    lam = C_LIGHT / (mhz * 1e6)
    radius = 0.22 * n / fov * lam
    r, t = radius * np.sqrt(rng.uniform(0, 1, N_ANT)), rng.uniform(0, 2 * math.pi, N_ANT)
    pair = np.array([(i, j) for i in range(N_ANT) for j in range(i + 1, N_ANT)])
    e, nn = (np.diff(a[pair], axis=1)[:, 0] for a in (r * np.cos(t), r * np.sin(t)))
    x, y, z = -math.sin(LAT) * nn, e, math.cos(LAT) * nn
    per_chan = -(-rows // chans)
    dumps = -(-per_chan // N_BASE)
    k = torch.arange(0, rows, every, device="cuda")
    chan, in_chan = k // per_chan, k % per_chan
    dump, base = in_chan // N_BASE, in_chan % N_BASE
    h = (-4.0 + 8.0 * dump.double() / max(1, dumps - 1)) * (15.0 * DEG)
    x, y, z = (torch.from_numpy(a).cuda()[base] for a in (x, y, z))
    sh, ch, sd, cd = torch.sin(h), torch.cos(h), math.sin(DEC), math.cos(DEC)
    scale = (1.0 + chan.double() / (mhz if chans > 1 else 1.0)) / lam  # 1 MHz channels
    return torch.stack([sh * x + ch * y, -sd * ch * x + sd * sh * y + cd * z, cd * ch * x - cd * sh * y + sd * z], 1) * scale[:, None]


def _stokes_uvw(case, seed):
    rng = _rng(seed, 12)
    r = 0.78 * case["n"] / 2 / case["fov"] * np.sqrt(rng.uniform(0, 1, case["rows"]))
    t = rng.uniform(0, 2 * math.pi, case["rows"])
    return torch.from_numpy(np.stack([r * np.cos(t), r * np.sin(t), rng.uniform(-200.0, 200.0, case["rows"])], 1)).cuda()


def _sources(seed, fov, count=6):
    rng = _rng(seed, 2)
    r, t = 0.2 * fov * np.sqrt(rng.uniform(0, 1, count)), rng.uniform(0, 2 * math.pi, count)
    i, p, chi, v = rng.uniform(0.1, 1, count), rng.uniform(0, 0.1, count), rng.uniform(0, math.pi, count), rng.uniform(-0.01, 0.01, count)
    return r * np.cos(t), r * np.sin(t), np.stack([i, p * i * np.cos(2 * chi), p * i * np.sin(2 * chi), v * i], 1)


def _vis(uvw, npol, fov, seed, salt=3):
    """Visibilities of a few polarised point sources with receiver noise, complex64 [rows][npol]."""
    l, m, iquv = _sources(seed, fov)
    g = _torch_gen(seed, salt)
    rows = uvw.shape[0]
    out = 0.05 * torch.view_as_complex(torch.randn((rows, npol, 2), device="cuda", generator=g))
    for a, b, s in zip(l, m, iquv):
        turns = uvw[:, 0] * a + uvw[:, 1] * b + uvw[:, 2] * (math.sqrt(1 - a * a - b * b) - 1)
        ph = torch.polar(torch.ones_like(turns), 2 * math.pi * torch.remainder(turns, 1.0)).to(torch.complex64)
        corr = [s[0]] if npol == 1 else [s[0] + s[1], complex(s[2], s[3]), complex(s[2], -s[3]), s[0] - s[1]]
        out += ph[:, None] * torch.tensor(corr, dtype=torch.complex64, device="cuda")
    return out


def _model(n, npol, fov, seed, count=50):
    """A component model, float32 [npol][n][n], in the inner half of the field."""
    rng = _rng(seed, 4)
    img = torch.zeros((npol, n, n), dtype=torch.float32, device="cuda")
    y, x = rng.integers(n // 4, 3 * n // 4, count), rng.integers(n // 4, 3 * n // 4, count)
    _, _, iquv = _sources(seed + 77, fov, count)
    img[:, torch.from_numpy(y).cuda(), torch.from_numpy(x).cuda()] = torch.from_numpy(iquv[:, :npol].T.astype(np.float32)).cuda()
    return img


def _geometry(n, planes, fov, os=8, mk=256, support=None, w_max=None):
    w_max = 0.34 * n / fov if w_max is None else w_max
    w = np.linspace(-w_max, w_max, planes) if planes > 1 else np.zeros(1)
    if support is None:
        s = np.clip(2 * np.ceil((7 + 0.8 * np.abs(w) * fov * fov) / 2.0), 16, 48).astype(np.int32)
    else:
        s = np.full(planes, support, np.int32)
    return SimpleNamespace(n=n, cell=fov / n, os=os, w_planes=w, support=s, tile=np.full(planes, 16, np.int32), aa_support=AA,
                           mk=mk, nplanes=planes, fov=fov)


def _jones(geom, mhz, seed):
    """Gaussian beam with 1 % leakage on the kernel lattice, complex128 [2][2][mk][mk]."""
    rng = _rng(seed, 5)
    theta = 1.0 * DEG * 1400.0 / mhz
    a, b = (rng.standard_normal((2, 3)) + 1j * rng.standard_normal((2, 3))) / math.sqrt(2.0)
    x = (np.arange(geom.mk) - geom.mk // 2) * (geom.fov / geom.mk)
    m, l = np.meshgrid(x, x, indexing="ij")
    e = np.exp(-2.0 * math.log(2.0) * (l * l + m * m) / theta**2)
    return np.stack([np.stack([e + 0j, e * 0.01 * (a[0] + a[1] * l / theta + a[2] * m / theta)]),
                     np.stack([e * 0.01 * (b[0] + b[1] * l / theta + b[2] * m / theta), e + 0j])])


def _field(case, seed, storage, mhz, rows, chans, directions, plan=True):
    """Tuned geometry, kernel sets and plan of a full-polarisation field, as the benchmark sets them up."""
    pg.use_torch_allocator(True)
    launch = autotune.apply(_geometry(case["n"], case["planes"], case["fov"]), 4, storage)
    jones = _jones(launch.geom, mhz, seed)
    s = SimpleNamespace(launch=launch, uvw=_uvw(rows, case["n"], case["fov"], mhz, chans, seed))
    s.kernels = {d: pg.make_kernels(launch.geom, 4, d, jones=jones, eps_null=0.2, storage=storage) for d in directions}
    s.plan = autotune.plan(s.kernels[directions[0]], s.uvw, launch) if plan else None
    return s


def _batch_fields(case, seed):
    rng = _rng(seed + 0, 6)
    f = case["fields"]
    rows = np.geomspace(case["rows_hi"], case["rows_lo"], f).astype(int)
    return [(int(r) + 13 * i, 700.0 + 1100.0 * i / max(1, f - 1), int(rng.integers(1 << 30))) for i, r in enumerate(rows)]


def _clean_inputs(case, seed):
    """A residual of point sources under a point-spread function with sidelobes, plus noise."""
    n, npol, rng = case["n"], case["npol"], _rng(seed, 7)
    x = torch.arange(n, device="cuda", dtype=torch.float64) - n // 2
    r2 = x[None, :] ** 2 + (x[:, None] * 1.1) ** 2
    psf = (torch.exp(-r2 / 8.0) + 0.06 * torch.cos(0.35 * x)[None, :] * torch.cos(0.21 * x)[:, None] * torch.exp(-r2 / (0.12 * n) ** 2))
    psf = (psf / psf[n // 2, n // 2]).float().contiguous()
    img = 1e-3 * torch.randn((npol, n, n), device="cuda", generator=_torch_gen(seed, 8))
    pos = rng.integers(n // 4, 3 * n // 4, (40, 2))
    _, _, iquv = _sources(seed, 0.06, 40)
    half = n // 4
    for (py, px), s in zip(pos, iquv):
        patch = psf[n // 2 - half:n // 2 + half, n // 2 - half:n // 2 + half]
        img[:, py - half:py + half, px - half:px + half] += torch.tensor(s[:npol], dtype=torch.float32, device="cuda")[:, None, None] * patch
    mask = (r2 < (0.42 * n) ** 2).to(torch.uint8).contiguous()
    return img, psf, mask


def _resample_inputs(case, seed):
    n, npol = case["n"], case["npol"]
    nm = 2 * int(n * case["pad"] / 2)
    cell = 0.065 / n
    g = _torch_gen(seed, 9)
    img = torch.randn((npol, n, n), device="cuda", generator=g)
    x = (torch.arange(n, device="cuda", dtype=torch.float64) - n // 2) * cell
    power = torch.exp(-4.0 * math.log(2.0) * (x[None, :] ** 2 + x[:, None] ** 2) / DEG**2)
    weight = torch.where(power >= 0.2, power**2, torch.zeros_like(power)).float().contiguous()
    base = torch.randn((npol, nm, nm), device="cuda", generator=g)
    base_w = torch.rand((nm, nm), device="cuda", generator=g)
    turn = float(_rng(seed, 10).uniform(0, 2 * math.pi))
    off = case["offset"] * DEG
    return img, weight, base, base_w, (n, cell, 1.0 + off * math.cos(turn) / math.cos(DEC), DEC + off * math.sin(turn)), (nm, cell, 1.0, DEC)


def _train_inputs(case, seed):
    g = _torch_gen(seed, 11)
    dims = [case["features"]] + [case["width"]] * case["hidden"] + [case["outputs"]]
    layers = [((2 * torch.rand((a, b), device="cuda", generator=g) - 1) * math.sqrt((6.0 if b != dims[-1] or i + 2 < len(dims) else 3.0) / a),
               0.01 * torch.randn(b, device="cuda", generator=g)) for i, (a, b) in enumerate(zip(dims[:-1], dims[1:]))]
    x = 2 * torch.rand((case["batch"], dims[0]), device="cuda", generator=g) - 1
    t = torch.randn((case["batch"], dims[-1]), device="cuda", generator=g) * torch.exp(-torch.arange(dims[-1], device="cuda") / 40.0)
    return dims, layers, x, t


# ----------------------------------------------------------------------------------- prepare and run

def _usable(kernels):
    """float32 [n][n]: one where the taper correction is well conditioned, as clean restricts itself to;
    towards the edge of the image it amplifies the rounding of the gridding sums without bound."""
    return clean.taper_mask(kernels).float()


def prepare(case, seed):
    kind = case["kind"]
    pg.use_torch_allocator(True)
    if kind == "stokes_step":
        geom = _geometry(case["n"], case["planes"], case["fov"], os=case["os"], mk=case["n"], support=case["support"], w_max=200.0)
        uvw = _stokes_uvw(case, seed)
        kernels = pg.make_kernels(geom, 1, pg.KIND_GRID)
        return SimpleNamespace(case=case, kernels=kernels, predict=pg.make_kernels(geom, 1, pg.KIND_DEGRID), uvw=uvw, usable=_usable(kernels),
                               vis=_vis(uvw, 1, case["fov"], seed), model=_model(case["n"], 1, case["fov"], seed, 5))
    if kind == "cycle":
        s = _field(case, seed, pg.STORE_F32, case["mhz"], case["rows"], case["chans"], (pg.KIND_GRID, pg.KIND_DEGRID), plan=case["keep_plan"])
        s.vis, s.model = _vis(s.uvw, 4, case["fov"], seed), _model(case["n"], 4, case["fov"], seed)
        s.residual, s.usable = torch.empty_like(s.vis), _usable(s.kernels[pg.KIND_GRID])
        s.grid = torch.empty((4, case["n"], case["n"]), dtype=torch.complex64, device="cuda")
    elif kind == "plan":
        s = _field(case, seed, pg.STORE_F32, case["mhz"], case["rows"], case["chans"], (pg.KIND_GRID,), plan=False)
        s.items = torch.zeros((case["rows"], 8), dtype=torch.int32, device="cuda")
    elif kind == "grid":
        s = _field(case, seed, case["storage"], case["mhz"], case["rows"], case["chans"], (pg.KIND_GRID,))
        s.vis = _vis(s.uvw, 4, case["fov"], seed)
        s.grid = torch.empty((4, case["n"], case["n"]), dtype=torch.complex64, device="cuda")
    elif kind == "degrid":
        s = _field(case, seed, case["storage"], case["mhz"], case["rows"], case["chans"], (pg.KIND_DEGRID,))
        s.grid = torch.fft.ifft2(_model(case["n"], 4, case["fov"], seed).to(torch.complex64), norm="forward")
        s.vis = torch.empty((case["rows"], 4), dtype=torch.complex64, device="cuda")
    elif kind == "batch":
        s = SimpleNamespace(fields=[])
        down, up = [], []
        launch = autotune.apply(_geometry(case["n"], case["planes"], case["fov"]), 4, pg.STORE_F16)
        for rows, mhz, sub in _batch_fields(case, seed):
            jones = _jones(launch.geom, mhz, sub)
            kg = pg.make_kernels(autotune.batch_grid_geom(launch), 4, pg.KIND_GRID, jones=jones, eps_null=0.2, storage=pg.STORE_F16)
            kd = pg.make_kernels(launch.geom, 4, pg.KIND_DEGRID, jones=jones, storage=pg.STORE_F16)
            uvw = _uvw(rows, case["n"], case["fov"], mhz, 1, sub)
            p, q = autotune.batch_plans(kg, kd, uvw, launch)
            vis, out = _vis(uvw, 4, case["fov"], sub), torch.empty((rows, 4), dtype=torch.complex64, device="cuda")
            grid = torch.empty((4, case["n"], case["n"]), dtype=torch.complex64, device="cuda")
            model = torch.fft.ifft2(_model(case["n"], 4, case["fov"], sub).to(torch.complex64), norm="forward")
            s.fields.append((p, kg, vis, grid, q, kd, out, model))
            down.append((p, kg, vis, grid))
            up.append((q, kd, out, model))
        s.down, s.up = pg.batch(down), pg.batch(up)
    elif kind == "kernels":
        geom = autotune.apply(_geometry(case["n"], case["planes"], case["fov"], mk=case["mk"]), 4, case["storage"]).geom
        s = SimpleNamespace(geom=geom, jones=_jones(geom, 1400.0, seed))
    elif kind == "clean":
        s = SimpleNamespace()
        s.dirty, s.psf, s.mask = _clean_inputs(case, seed)
    elif kind == "resample":
        s = SimpleNamespace()
        s.img, s.weight, s.base, s.base_w, s.field, s.mosaic = _resample_inputs(case, seed)
        s.acc, s.acc_w, s.back = torch.empty_like(s.base), torch.empty_like(s.base_w), torch.empty_like(s.img)
    else:
        dims, layers, x, t = _train_inputs(case, seed)
        s = SimpleNamespace(net=pg.MLP(dims[0], case["width"], case["hidden"], dims[-1], case["batch"], seed=1), x=x, t=t)
        for i, (w, b) in enumerate(layers):
            s.net.load(i, w, b)
    s.case = case
    return s


def run(state):
    s, case = state, state.case
    kind = case["kind"]
    if kind == "stokes_step":
        p = pg.plan(s.kernels, s.uvw)
        return {"image": pg.image(p, s.kernels, s.vis, float(case["rows"])).mul_(s.usable), "vis": pg.predict(p, s.predict, s.model)}
    if kind == "cycle":
        p = s.plan if s.plan is not None else autotune.plan(s.kernels[pg.KIND_GRID], s.uvw, s.launch)
        img = pg.image(p, s.kernels[pg.KIND_GRID], s.vis, float(case["rows"]), grid_buf=s.grid).mul_(s.usable)
        s.residual.copy_(s.vis)
        return {"image": img, "residual": pg.predict(p, s.kernels[pg.KIND_DEGRID], s.model, out=s.residual, buf=s.grid, subtract=True)}
    if kind == "plan":
        perm, fine, items = autotune.plan(s.kernels[pg.KIND_GRID], s.uvw, s.launch).arrays()
        s.items[:items.shape[0]] = items
        return [perm, fine, s.items]
    if kind == "grid":
        return pg.grid(s.plan, s.kernels[pg.KIND_GRID], s.vis, out=s.grid, fftshift=True, deterministic=case["exactly"])
    if kind == "degrid":
        return pg.degrid(s.plan, s.kernels[pg.KIND_DEGRID], s.grid, out=s.vis, fftshift=True)
    if kind == "batch":
        s.down.grid(fftshift=True)
        s.up.degrid(fftshift=True)
        return {"grids": [f[3] for f in s.fields], "vis": [f[6] for f in s.fields]}
    if kind == "kernels":
        return pg.make_kernels(s.geom, 4, case["direction"], jones=s.jones, eps_null=0.2, storage=case["storage"]).table()
    if kind == "clean":
        residual, model = s.dirty.clone(), torch.zeros_like(s.dirty)
        pos, val = pg.hogbom(residual, s.psf, s.mask, gain=0.1, threshold=1e-4, max_iter=case["iters"], psf_patch=case["patch"], model=model)
        return {"pos": pos, "val": val, "residual": residual, "model": model}
    if kind == "resample":
        s.acc.copy_(s.base)
        s.acc_w.copy_(s.base_w)
        pg.reproject(s.img, s.field, s.acc, s.mosaic, src_weight=s.weight, dst_weight=s.acc_w, accumulate=True)
        pg.weight_normalise(s.acc, s.acc_w, 0.05)
        return {"mosaic": s.acc, "weight": s.acc_w, "field": pg.reproject(s.acc, s.mosaic, s.back, s.field)}
    loss = s.net.train_step(s.x, s.t, 1e-3)
    return {"loss": loss, "weights": [s.net.copy(pg.MLP_W, i) for i in range(case["hidden"] + 1)]}


# ------------------------------------------------------------------------------------------- the work

def _taps(case, rows, mhz, chans, seed=0):
    """Sum over rows of the squared support, from a thinned draw of the tracks."""
    geom = _geometry(case["n"], case["planes"], case["fov"])
    w = _uvw(rows, case["n"], case["fov"], mhz, chans, seed, every=max(1, rows // 20000))[:, 2].cpu().numpy()
    p = np.abs(w[:, None] - geom.w_planes[None, :]).argmin(1)
    return float((geom.support[p].astype(np.float64) ** 2).mean()) * rows, 64.0 * 16 * float((geom.support.astype(np.float64) ** 2).sum())


def work(case):
    kind = case["kind"]
    if kind == "stokes_step":
        rows, pix = case["rows"], float(case["n"]) ** 2
        table = case["planes"] * case["os"] ** 2 * case["support"] ** 2 * 8.0
        return dict(flops=16.0 * case["support"] ** 2 * rows + 2 * 10 * pix * math.log2(case["n"]),
                    bytes=rows * (24 + 8 + 8) + 2 * table + pix * (4 + 4 + 4 * 8 * 2))
    if kind == "cycle":
        rows, pix = case["rows"], float(case["n"]) ** 2
        taps, entries = _taps(case, rows, case["mhz"], case["chans"])
        return dict(flops=2 * 128.0 * taps + 2 * 4 * 10 * pix * math.log2(case["n"]),
                    bytes=rows * (32 + 64 + 24) + 2 * 8 * entries + 4 * pix * (8 + 16 + 12 + 12 + 16 + 8))
    if kind == "plan":
        return dict(flops=0.0, bytes=case["rows"] * (24.0 + 4 + 8))
    if kind in ("grid", "degrid"):
        taps, entries = _taps(case, case["rows"], case["mhz"], case["chans"])
        return dict(flops=128.0 * taps, bytes=case["rows"] * (12 + 32.0) + entries * (4 if case["storage"] else 8) + 32.0 * case["n"] ** 2)
    if kind == "batch":
        flops = byts = 0.0
        for rows, mhz, sub in _batch_fields(case, 0):
            taps, entries = _taps(case, rows, mhz, 1, sub)
            flops += 2 * 128.0 * taps
            byts += 2 * (rows * (12 + 32.0) + entries * 4 + 32.0 * case["n"] ** 2)
        return dict(flops=flops, bytes=byts)
    if kind == "kernels":
        s = _geometry(case["n"], case["planes"], case["fov"]).support.astype(np.float64) * 8
        mk = float(case["mk"])
        return dict(flops=float(16 * 8 * (mk * mk * s + s * s * mk).sum()), bytes=float(16 * (s * s).sum()) * (4 if case["storage"] else 8) + 64 * mk * mk)
    if kind == "clean":
        side = min(case["n"], 2 * case["patch"] + 1)
        pix = float(case["n"]) ** 2
        return dict(flops=2.0 * case["iters"] * case["npol"] * side * side,
                    bytes=pix * (1 + 4 + case["npol"] * 16) + case["iters"] * side * side * (4 + 8.0 * case["npol"]))
    if kind == "resample":
        pix, mos = float(case["n"]) ** 2, float(2 * int(case["n"] * case["pad"] / 2)) ** 2
        return dict(flops=8.0 * case["npol"] * (pix + mos), bytes=case["npol"] * (4 * pix * 2 + 4 * mos * 4) + 4 * pix + 8 * mos)
    dims = [case["features"]] + [case["width"]] * case["hidden"] + [case["outputs"]]
    params = sum(a * b for a, b in zip(dims[:-1], dims[1:]))
    return dict(flops=6.0 * params * case["batch"], bytes=params * (7 * 4 + 4.0) + 4.0 * case["batch"] * (dims[0] + dims[-1]))


# ---------------------------------------------------------------------------------- the same in 64 bits

def _spheroidal(x):
    """The order-0 prolate spheroidal function of c = pi AA / 2, one at x = 0, by its Legendre expansion."""
    c, m = math.pi * AA / 2.0, 60
    k = 2.0 * np.arange(m)
    a = np.diag(k * (k + 1) + c * c * (2 * k * (k + 1) - 1) / ((2 * k + 3) * (2 * k - 1)))
    off = c * c * (k + 2) * (k + 1) / ((2 * k + 3) * np.sqrt((2 * k + 1) * (2 * k + 5)))
    a += np.diag(off[:-1], 1) + np.diag(off[:-1], -1)
    coef = np.zeros(2 * m)
    coef[::2] = np.linalg.eigh(a)[1][:, 0] * np.sqrt(k + 0.5)
    return np.polynomial.legendre.legval(x, coef) / np.polynomial.legendre.legval(0.0, coef)


def _screens(geom, jones, direction):
    """Mueller screens complex128 [4][4][mk][mk]: the regularised inverse, or the predicting adjoint."""
    if jones is None:
        return torch.ones((1, 1, geom.mk, geom.mk), dtype=torch.complex128, device="cuda")
    j = torch.from_numpy(jones).cuda().permute(2, 3, 0, 1)
    s = torch.tensor([[0.5, 0, 0, 0.5], [0.5, 0, 0, -0.5], [0, 0.5, 0.5, 0], [0, -0.5j, 0.5j, 0]], dtype=torch.complex128, device="cuda")
    ms = (j[:, :, :, None, :, None] * j.conj()[:, :, None, :, None, :]).reshape(geom.mk, geom.mk, 4, 4)
    ms = s @ ms @ torch.linalg.inv(s)
    if direction == pg.KIND_DEGRID:
        phi = (torch.linalg.inv(s) @ ms).conj().transpose(-1, -2)
    else:
        b = torch.diagonal(ms, dim1=-2, dim2=-1).clone()
        beta = (0.2 / 2 * b.abs().amax((0, 1))) ** 2
        ms = ms + torch.diag_embed(b * beta / b.abs() ** 2)
        phi = torch.linalg.inv(ms) @ s
    return phi.permute(2, 3, 0, 1).contiguous()


def _plane_table(geom, p, phi):
    """Plane p's oversampled kernels complex128 [q][c][os][os][S][S] (phase y, phase x, tap y, tap x)."""
    mk, s, os = geom.mk, int(geom.support[p]), geom.os
    a = np.arange(mk) - mk // 2
    aa = torch.from_numpy(_spheroidal(2.0 * a / mk)).cuda()
    l = torch.from_numpy(a * (geom.fov / mk)).cuda()
    r2 = l[None, :] ** 2 + l[:, None] ** 2
    turns = geom.w_planes[p] * (-r2 / (1.0 + torch.sqrt(1.0 - r2)))
    f = phi * torch.polar(aa[:, None] * aa[None, :], -2 * math.pi * torch.remainder(turns, 1.0))
    d = np.arange(s * os) - (s * os // 2 - 1)
    e = np.exp(2j * math.pi * ((d[:, None] * a[None, :]) % (os * mk)) / (os * mk)) / mk
    e[-1] = 0.0
    e = torch.from_numpy(e).cuda()
    t = e @ (f @ e.T)
    q, c = t.shape[:2]
    return t.reshape(q, c, s, os, s, os).permute(0, 1, 3, 5, 2, 4)


def _stored(t, storage):
    if storage == pg.STORE_F16:
        return torch.view_as_complex(torch.view_as_real(t.contiguous()).half().double())
    return t.to(torch.complex64).to(torch.complex128)


def _binned(geom, uvw):
    """Plane, footprint corner (y, x) and kernel phase of every row, and whether it is kept."""
    fine = torch.floor((uvw[:, :2] * (geom.n * geom.cell) + geom.n / 2.0) * geom.os + 0.5).long()
    w = torch.from_numpy(np.asarray(geom.w_planes)).cuda()
    plane = torch.cat([(u[:, None] - w[None, :]).abs().argmin(1) for u in uvw[:, 2].split(1 << 20)])
    s = torch.from_numpy(np.asarray(geom.support)).cuda().long()[plane]
    half = s * geom.os // 2
    corner = -torch.div(-(fine - half[:, None] + 1), geom.os, rounding_mode="floor")
    phase = corner * geom.os - fine + half[:, None] - 1
    kept = (corner >= 0).all(1) & (corner + s[:, None] <= geom.n).all(1)
    return plane, corner, phase[:, 1] * geom.os + phase[:, 0], kept


def _by_plane(geom, jones, direction, storage, uvw):
    """For each plane with rows, in parts: (table [phase][tap][q][c], rows, phases, pixel of every tap)."""
    plane, corner, phase, kept = _binned(geom, uvw)
    phi = _screens(geom, jones, direction)
    for p in range(geom.nplanes):
        rows = torch.nonzero((plane == p) & kept)[:, 0]
        if not len(rows):
            continue
        s = int(geom.support[p])
        t = _stored(_plane_table(geom, p, phi), storage)
        t = t.permute(2, 3, 4, 5, 0, 1).reshape(geom.os**2, s * s, t.shape[0], t.shape[1]).contiguous()
        tap = torch.arange(s * s, device="cuda")
        step = (tap // s) * geom.n + tap % s
        for r in rows.split(max(1, (1 << 22) // (s * s))):
            yield t, r, phase[r], (corner[r, 1] * geom.n + corner[r, 0])[:, None] + step


def _grid64(geom, jones, storage, uvw, vis, shift=True):
    npol = vis.shape[1]
    out = torch.zeros((geom.n * geom.n, npol, 2), dtype=torch.float64, device="cuda")
    v = vis.to(torch.complex128)
    for t, r, ph, pix in _by_plane(geom, jones, pg.KIND_GRID, storage, uvw):
        y = (t[ph] * v[r][:, None, None, :]).sum(-1)
        out.index_add_(0, pix.reshape(-1), torch.view_as_real(y).reshape(-1, npol, 2))
    g = torch.view_as_complex(out).T.reshape(npol, geom.n, geom.n)
    return g * _checker(geom.n) if shift else g


def _checker(n):
    a = 1.0 - 2.0 * (torch.arange(n, device="cuda") % 2).double()
    return a[:, None] * a[None, :]


def _degrid64(geom, jones, storage, uvw, grid):
    npol = grid.shape[0]
    g = (grid.to(torch.complex128) * _checker(geom.n)).reshape(npol, -1).T.contiguous()
    out = torch.zeros((uvw.shape[0], npol), dtype=torch.complex128, device="cuda")
    for t, r, ph, pix in _by_plane(geom, jones, pg.KIND_DEGRID, storage, uvw):
        out[r] = (t[ph].conj() * g[pix][..., None]).sum((1, 2))
    return out


def _taper64(geom):
    aa = torch.from_numpy(_spheroidal(2.0 * (np.arange(geom.n) - geom.n // 2) / geom.n)).cuda()
    return _checker(geom.n) / (aa[:, None] * aa[None, :])


def _cycle64(geom, jones, uvw, vis, model, rows):
    img = (torch.fft.fft2(_grid64(geom, jones, pg.STORE_F32, uvw, vis)) * _taper64(geom)).real / rows
    img *= _taper64(geom).abs() <= 10.0
    g = torch.fft.ifft2((model.double() * _taper64(geom)).to(torch.complex128), norm="forward")
    return img, _degrid64(geom, jones, pg.STORE_F32, uvw, g)


def _clean64(case, seed):
    img, psf, mask = _clean_inputs(case, seed)
    n, patch = case["n"], case["patch"]
    gain, threshold = float(np.float32(0.1)), float(np.float32(1e-4))
    r, psf, model, vals = img.double(), psf.double(), torch.zeros_like(img).double(), []
    for _ in range(case["iters"]):
        score = torch.where(mask > 0, r[0].abs(), -1.0).reshape(-1)
        at = int(score.argmax())
        if float(score[at]) < threshold:
            break
        py, px = divmod(at, n)
        v = gain * r[:, py, px]
        vals.append(v)
        model[:, py, px] += v
        y0, y1 = max(0, py - n // 2, py - patch), min(n, py + n // 2, py + patch + 1)
        x0, x1 = max(0, px - n // 2, px - patch), min(n, px + n // 2, px + patch + 1)
        r[:, y0:y1, x0:x1] -= v[:, None, None] * psf[y0 - py + n // 2:y1 - py + n // 2, x0 - px + n // 2:x1 - px + n // 2]
    return {"pos": None, "val": torch.stack(vals), "residual": r, "model": model}


def _resample64(src, weight, sf, df):
    """Bilinear samples of src (and weight) at the pixels of frame df: values, weights."""
    def axes(f):
        _, _, ra, dec = f
        sa, ca, sd, cd = math.sin(ra), math.cos(ra), math.sin(dec), math.cos(dec)
        return np.array([[-sa, ca, 0.0], [-sd * ca, -sd * sa, cd], [cd * ca, cd * sa, sd]])
    rot = axes(sf) @ axes(df).T
    x = (torch.arange(df[0], device="cuda", dtype=torch.float64) - df[0] // 2) * df[1]
    l0, m0 = x[None, :].expand(df[0], df[0]), x[:, None].expand(df[0], df[0])
    d = torch.stack([l0, m0, torch.sqrt(1.0 - l0 * l0 - m0 * m0)], -1) @ torch.from_numpy(rot.T.copy()).cuda()
    px, py, top = d[..., 0] / sf[1] + sf[0] // 2, d[..., 1] / sf[1] + sf[0] // 2, sf[0] - 1
    inside = (d[..., 2] > 0) & (px >= -1e-6) & (py >= -1e-6) & (px <= top + 1e-6) & (py <= top + 1e-6)
    px, py = px.clamp(0, top), py.clamp(0, top)
    x0, y0 = px.floor().clamp(max=top - 1).long(), py.floor().clamp(max=top - 1).long()
    fx, fy = px - x0, py - y0

    def sample(a):
        a = a.double()
        v = (1 - fy) * ((1 - fx) * a[..., y0, x0] + fx * a[..., y0, x0 + 1]) + fy * ((1 - fx) * a[..., y0 + 1, x0] + fx * a[..., y0 + 1, x0 + 1])
        return torch.where(inside, v, 0.0)
    return sample(src), sample(weight) if weight is not None else inside.double()


def _train64(case, seed):
    """One Adam step in 64 bits from the same weights."""
    _, layers, x, t = _train_inputs(case, seed)
    ws = [w.double().requires_grad_() for w, _ in layers]
    h, t = x.double(), t.double()
    for i, w in enumerate(ws):
        h = h @ w + layers[i][1].double()
        if i + 1 < len(ws):
            h = torch.nn.functional.silu(h)
    loss = ((h - t).square().sum(1) / t.square().sum(1)).mean()
    grads = torch.autograd.grad(loss, ws)
    return {"loss": loss.detach().reshape(1), "weights": [(w - 1e-3 * g / (g.abs() + 1e-8)).detach() for w, g in zip(ws, grads)]}


def exact(case, seed):
    kind = case["kind"]
    if kind == "plan":
        return None
    if kind == "stokes_step":
        geom = _geometry(case["n"], case["planes"], case["fov"], os=case["os"], mk=case["n"], support=case["support"], w_max=200.0)
        uvw = _stokes_uvw(case, seed)
        img, vis = _cycle64(geom, None, uvw, _vis(uvw, 1, case["fov"], seed), _model(case["n"], 1, case["fov"], seed, 5), case["rows"])
        return {"image": img, "vis": vis}
    if kind in ("cycle", "grid", "degrid"):
        geom = _geometry(case["n"], case["planes"], case["fov"])
        jones = _jones(geom, case["mhz"], seed)
        uvw = _uvw(case["rows"], case["n"], case["fov"], case["mhz"], case["chans"], seed)
        model = _model(case["n"], 4, case["fov"], seed)
        if kind == "degrid":
            return _degrid64(geom, jones, case["storage"], uvw, torch.fft.ifft2(model.to(torch.complex64), norm="forward"))
        vis = _vis(uvw, 4, case["fov"], seed)
        if kind == "grid":
            return _grid64(geom, jones, case["storage"], uvw, vis)
        img, pred = _cycle64(geom, jones, uvw, vis, model, case["rows"])
        return {"image": img, "residual": vis.to(torch.complex128) - pred}
    if kind == "batch":
        geom, grids, viss = _geometry(case["n"], case["planes"], case["fov"]), [], []
        for rows, mhz, sub in _batch_fields(case, seed):
            jones, uvw = _jones(geom, mhz, sub), _uvw(rows, case["n"], case["fov"], mhz, 1, sub)
            grids.append(_grid64(geom, jones, pg.STORE_F16, uvw, _vis(uvw, 4, case["fov"], sub)))
            model = torch.fft.ifft2(_model(case["n"], 4, case["fov"], sub).to(torch.complex64), norm="forward")
            viss.append(_degrid64(geom, jones, pg.STORE_F16, uvw, model))
        return {"grids": grids, "vis": viss}
    if kind == "kernels":
        geom = _geometry(case["n"], case["planes"], case["fov"], mk=case["mk"])
        phi = _screens(geom, _jones(geom, 1400.0, seed), case["direction"])
        e = 4 if case["storage"] else 2  # the table: [phase y][phase x][chunk][tap y][tap x][entry], chunks of 16 bytes
        parts = []
        for p in range(geom.nplanes):
            t = _plane_table(geom, p, phi)
            s = t.shape[-1]
            parts.append(t.reshape(16 // e, e, 8, 8, s, s).permute(2, 3, 0, 4, 5, 1).reshape(-1))
        t = torch.cat(parts)
        return torch.view_as_real(t) if case["storage"] else t
    if kind == "clean":
        return _clean64(case, seed)
    if kind == "resample":
        img, weight, base, base_w, field, mosaic = _resample_inputs(case, seed)
        v, w = _resample64(img, weight, field, mosaic)
        total = base_w.double() + w
        acc = torch.where(total >= 0.05, (base.double() + w * v) / total, 0.0)
        return {"mosaic": acc, "weight": total, "field": _resample64(acc, None, mosaic, field)[0]}
    return _train64(case, seed)

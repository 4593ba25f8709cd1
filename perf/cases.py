"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values; its "kind" names the program:

  lattice   one D2Q9 lattice (``Lattice``): advance it by some steps, then read
            the fields and the force records of those steps
  batch     many uneven channels (``LatticeBatch``): one interval between two
            checks, then the status and every case's fields
  tube      one D3Q19 lattice (``Lattice3D``): as lattice, a tube with a sphere
  train     one training step of the warm-start network, gradients read
  infer     warm-start fields of a batch of channels and their start check

``exact`` gives the same outputs in 64 bits: the lattice Boltzmann step and
the network written out in plain torch from their equations.
"""
import math
import os

import numpy as np
import torch

import lbm_cases
import paper_1303_0625_amd as pkg
from paper_1303_0625_amd import lbm, warmstart

BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
LARGEST = 50 * 4096 * 4096  # node updates of the largest listed lattice


# ------------------------------------------------------------------ the cases
def _lattice(**kw):
    c = {"kind": "lattice", "nx": 128, "ny": 64, "walls": True, "dtype": "f32", "fixed": 0, "moving": 0, "free": False,
         "interpolated": False, "mrt": False, "refill": 0, "steps": 1}
    c.update(kw)
    return c


def _tube(**kw):
    c = {"kind": "tube", "nx": 150, "n": 42, "dtype": "f32", "pressure": False, "interpolated": False, "free": False,
         "steps": 1}
    c.update(kw)
    return c


def listed():
    return [
        # the FP64 validation channel, a few steps at a time (a program that looks at the force as it goes):
        # launches and latency
        dict(_lattice(nx=128, ny=64, dtype="f64", fixed=1, steps=8), name="channel_128x64_f64"),
        # a channel with fixed and translating cylinders: refill, link rebuild, a cache-resident state
        dict(_lattice(nx=2048, ny=1024, fixed=16, moving=16, steps=100), name="moving_2048x1024_f32"),
        # the headline lattice: the largest, streamed from HBM
        dict(_lattice(nx=4096, ny=4096, walls=False, fixed=64, steps=50), name="periodic_4096_f32"),
        # the same in reduced-precision storage
        dict(_lattice(nx=4096, ny=4096, walls=False, fixed=64, dtype="f16", steps=50), name="periodic_4096_f16"),
        # a ragged channel with the operator and the boundary rule the paper simulates with
        dict(_lattice(nx=1001, ny=517, fixed=6, moving=6, interpolated=True, mrt=True, steps=64),
             name="ibb_mrt_1001x517_f32"),
        # a particle settling in a channel (the paper's sedimentation)
        dict(_lattice(nx=1200, ny=120, dtype="f64", free=True, interpolated=True, steps=100),
             name="sediment_1200x120_f64"),
        # uneven channels solved together (training data, parameter studies)
        {"kind": "batch", "cases": 64, "dtype": "f32", "steps": 100, "name": "batch_64_f32"},
        # the paper's tube: pressure planes, interpolated walls, a sphere at rest
        dict(_tube(pressure=True, interpolated=True, steps=100), name="tube_150x42_pressure"),
        # the same tube with the sphere free to migrate
        dict(_tube(interpolated=True, free=True, steps=32), name="tube_150x42_free"),
        # a tube streamed from HBM
        dict(_tube(nx=512, n=128, steps=50), name="tube_512x128"),
        # training and inference of the warm-start network at its shipped size
        {"kind": "train", "batch": 8, "name": "train_batch8"},
        {"kind": "infer", "batch": 32, "name": "infer_batch32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fixed", "fixed", "fixed", "moving", "moving", "free", "batch", "tube", "tube", "train", "infer"])
    if kind == "train":
        return {"kind": "train", "batch": _log(rng, 1, 32)}
    if kind == "infer":
        return {"kind": "infer", "batch": _log(rng, 1, 64)}
    if kind == "batch":
        return {"kind": "batch", "cases": rng.randint(4, 64), "dtype": rng.choice(["f32", "f32", "f16", "f64"]),
                "steps": 2 * rng.randint(10, 50)}
    if kind == "tube":
        n = _log(rng, 24, 128)
        free = rng.random() < 0.3
        nx = _log(rng, 2 * n, 4 * n)
        c = _tube(nx=nx, n=n, dtype=rng.choice(["f32", "f64"]), interpolated=rng.random() < 0.5, free=free,
                  pressure=not free and rng.random() < 0.5, steps=_log(rng, 4, 100))
        c["steps"] = max(2, min(c["steps"], LARGEST // (4 * nx * n * n), 16 if free else 100))
        return c
    walls = kind == "free" or rng.random() < 0.6
    if kind == "free":
        c = _lattice(nx=_log(rng, 300, 1500), ny=rng.randint(90, 240), walls=True, dtype="f64", free=True,
                     interpolated=rng.random() < 0.5, steps=_log(rng, 8, 100))
    else:
        nx, ny = _log(rng, 64, 4096), _log(rng, 64, 4096)
        room = max(1, nx * ny // 8192)
        mov = kind == "moving"
        nx, ny = (max(nx, 128), max(ny, 128)) if mov else (nx, ny)
        c = _lattice(nx=nx, ny=ny, walls=walls, dtype=rng.choice(["f32", "f32", "f64", "f16", "bf16"]),
                     fixed=min(32, rng.randint(1, room)), moving=min(16, max(1, min(room, ny // 64) // 2)) if mov else 0,
                     interpolated=rng.random() < 0.3, mrt=rng.random() < 0.3, refill=rng.randint(0, 2),
                     steps=_log(rng, 1, 100))
    c["steps"] = max(1, min(c["steps"], LARGEST // (c["nx"] * c["ny"])))
    return c


# ------------------------------------------------------------------ inputs
def _discs(rng, nx, ny, walls, fixed, moving):
    """Fixed discs with gaps of at least 5 nodes, and movers along x in horizontal lanes of their own."""
    bodies, lanes = [], []
    top = min(12.0, ny / 10.0, nx / 10.0)
    for _ in range(moving):
        r = float(rng.uniform(0.5 * top, top))
        for _ in range(5000):
            cy = float(rng.uniform(r + 8.0, ny - 9.0 - r))
            if all(cy - r - 5 > hi or cy + r + 5 < lo for lo, hi in lanes):
                break
        else:
            continue
        lanes.append((cy - r - 5, cy + r + 5))
        v = float(rng.uniform(0.01, 0.05)) * (1.0 if rng.uniform() < 0.5 else -1.0)
        bodies.append(lbm_cases.disc(float(rng.uniform(0, nx)), cy, r, vx=v, moves=True))
    placed = []
    for _ in range(fixed):
        r = float(rng.uniform(0.5 * top, top))
        for _ in range(5000):
            cx, cy = float(rng.uniform(0, nx)), float(rng.uniform(r + 6.0, ny - 7.0 - r))
            if any(cy - r <= hi and cy + r >= lo for lo, hi in lanes):
                continue
            if all(math.hypot(min(abs(cx - b["cx"]), nx - abs(cx - b["cx"])), cy - b["cy"]) - r - b["r"] >= 5
                   for b in placed):
                placed.append(lbm_cases.disc(cx, cy, r))
                break
    return bodies + placed


def _lattice_case(case, seed):
    rng = np.random.default_rng([seed, case["nx"], case["ny"]])
    nx, ny, walls = case["nx"], case["ny"], case["walls"]
    if case["free"]:
        r = ny / 8.0
        bodies = [lbm_cases.disc(float(rng.uniform(80, nx - 80)), float(rng.uniform(1.4, 1.8)) * r, r, moves=True)]
        return lbm_cases.make_case(nx, ny, 0.6, walls_y=True, bodies=bodies, refill=case["refill"]), rng
    bodies = _discs(rng, nx, ny, walls, case["fixed"], case["moving"])
    return lbm_cases.make_case(nx, ny, 0.6 if case["dtype"] != "f64" else 0.8, walls_y=walls, gx=1e-6, bodies=bodies,
                               refill=case["refill"]), rng


def _flow(rng, nx, ny, device):
    """A smooth flow: density and divergence-free velocity from a few Fourier modes (|u| up to about 0.03)."""
    x = torch.arange(nx, dtype=torch.float64, device=device) * (2 * math.pi / nx)
    y = torch.arange(ny, dtype=torch.float64, device=device) * (2 * math.pi / ny)
    rho = torch.ones((ny, nx), dtype=torch.float64, device=device)
    ux, uy = torch.full_like(rho, 0.01), torch.zeros_like(rho)
    for _ in range(3):
        kx, ky = int(rng.integers(1, 4)), int(rng.integers(1, 4))
        px, py, a = rng.uniform(0, 2 * math.pi), rng.uniform(0, 2 * math.pi), 0.008 * rng.uniform(0.5, 1.0)
        s = a / max(kx / nx, ky / ny)
        sx, cx, sy, cy = (torch.sin(kx * x + px), torch.cos(kx * x + px), torch.sin(ky * y + py), torch.cos(ky * y + py))
        ux += s * (ky / ny) * cy[:, None] * sx[None, :]
        uy -= s * (kx / nx) * sy[:, None] * cx[None, :]
        rho += 5e-4 * rng.uniform(0.5, 1.0) * sy[:, None] * cx[None, :]
    return rho, ux, uy


SED_RHO, SED_G = 1.03, 4.03e-4  # density of the settling disc and gravity along the channel


def _fields_dtype(case):
    return "f64" if case["dtype"] == "f64" else "f32"


def _lattice_inputs(case, seed, device):
    lc, rng = _lattice_case(case, seed)
    flow = None
    if not case["free"]:
        flow = _flow(rng, case["nx"], case["ny"], device)
        if _fields_dtype(case) == "f32":
            flow = tuple(a.float() for a in flow)
    return lc, flow


def _tube_case(case, seed):
    rng = np.random.default_rng([seed, case["nx"], case["n"]])
    nx, n = case["nx"], case["n"]
    R = 19.34 / 42.0 * n  # the paper's ratios
    r = 5.9 / 19.34 * R
    cy = (n - 1) / 2.0
    th = rng.uniform(0, 2 * math.pi)
    off = 0.21 * R
    sphere = dict(cx=float(nx * rng.uniform(0.25, 0.5)), cy=cy + off * math.cos(th), cz=cy + off * math.sin(th), r=r,
                  moves=case["free"])
    u0 = 0.0 if case["pressure"] else float(rng.uniform(0.005, 0.015))
    return dict(nx=nx, ny=n, nz=n, tau=0.6, duct=lbm.LBM3D_TUBE, R=R, u0=(u0, 0.0, 0.0),
                g=(0.0, 0.0, 0.0) if case["pressure"] else (1.825e-5 / nx, 0.0, 0.0), spheres=[sphere])


def _batch_cases(case, seed):
    """Channels of the benchmark's uneven sizes, the cylinder and the Reynolds number of each from the seed."""
    rng = np.random.default_rng([seed, case["cases"]])
    out = []
    for c in lbm_cases.uneven_channels(n_cases=case["cases"]):
        nx, ny = c["nx"], c["ny"]
        r = float(rng.uniform(0.05, 0.10) * ny)
        tau, g, _ = lbm_cases.re_to_tau_g(float(rng.uniform(1.0, 100.0)), 2 * r, ny)
        body = lbm_cases.disc(float(rng.uniform(0.25, 0.5) * nx), (ny - 1) / 2.0 + float(rng.uniform(-0.1, 0.1) * ny), r)
        out.append(lbm_cases.make_case(nx, ny, tau, walls_y=True, gx=g, bodies=[body]))
    return out


DROP = 1.5 * 1.825e-5  # half the pressure drop, as a density difference
TUBE_RHO = 1.2         # density of the free sphere

H, W, CH = 128, 256, (32, 64, 128, 256)


def _samples(seed, n, device):
    """n channels of the warm-start set with smooth stand-ins of their steady fields."""
    cs = lbm_cases.warmstart_channels(seed=seed, n_cases=n)
    rng = np.random.default_rng([seed, n])
    yy, xx = np.mgrid[0:H, 0:W]
    solid = np.zeros((n, H, W), np.uint8)
    for k, c in enumerate(cs):
        for b in c["bodies"]:
            solid[k] |= ((xx - b["cx"]) ** 2 + (yy - b["cy"]) ** 2 <= b["r"] ** 2).astype(np.uint8)
    g, tau = np.array([c["gx"] for c in cs]), np.array([c["tau"] for c in cs])
    uc = g * H * H / (8.0 * (tau - 0.5) / 3.0)
    ph = rng.uniform(0, 2 * math.pi, (n, 1, 1))
    wave = np.sin(2 * math.pi * xx / W + ph)
    prof = 1.0 - ((yy - (H - 1) / 2.0) / (H / 2.0)) ** 2
    fl = 1.0 - solid
    u = uc[:, None, None]
    ux, uy = fl * u * prof * (0.7 + 0.2 * wave), fl * u * 0.1 * prof * np.cos(2 * math.pi * xx / W + ph)
    rho = 1.0 + fl * u * 0.01 * wave
    d = {"solid": solid, "rho": rho.astype(np.float32), "ux": ux.astype(np.float32), "uy": uy.astype(np.float32),
         "re": np.array([c["Re"] for c in cs]), "gx": g, "tau": tau}
    return {k: torch.from_numpy(np.ascontiguousarray(v)).to(device) for k, v in d.items()}


RHO_SCALE = 0.01


def _params(case, seed):
    """Inference takes the shipped weights, training starts from random ones."""
    if case["kind"] == "infer":
        path = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "weights", "warmstart_256x128.npz")
        params, scale, _, _, _ = warmstart.load_weights(path)
        return torch.from_numpy(np.asarray(params, np.float32)), float(scale)
    return torch.from_numpy(warmstart.init_params(seed)), RHO_SCALE


def prepare(case, seed):
    kind = case["kind"]
    if kind == "lattice":
        lc, flow = _lattice_inputs(case, seed, "cuda")
        lat = pkg.Lattice(lc, dtype=case["dtype"], history_steps=case["steps"],
                          mrt=lbm.PAPER_MRT_RATES if case["mrt"] else None)
        if case["interpolated"]:
            lat.set_boundary(True)
        if case["free"]:
            lat.set_free(1, SED_RHO)
            lat.set_gravity((SED_G, 0.0), lbm.LBM_GME)
        else:
            lat.init_fields(*flow)
        return {"case": case, "lat": lat}
    if kind == "batch":
        b = pkg.LatticeBatch(_batch_cases(case, seed), dtype=case["dtype"])
        b.set_tiling(4, True)
        for k in range(b.n):
            b.init_poiseuille(k)
        return {"case": case, "batch": b}
    if kind == "tube":
        lat = pkg.Lattice3D(_tube_case(case, seed), dtype=case["dtype"], history_steps=case["steps"])
        if case["pressure"]:
            lat.set_pressure(1 + DROP, 1 - DROP)
        if case["interpolated"]:
            lat.set_boundary(True)
        if case["free"]:
            lat.set_free(1, TUBE_RHO)
        return {"case": case, "lat": lat}
    params, scale = _params(case, seed)
    net = pkg.WarmStartNet(H, W, case["batch"], dtype="bf16", ch=CH, rho_scale=scale)
    net.set_params(params)
    state = {"case": case, "net": net, "data": _samples(seed, case["batch"], "cuda")}
    if kind == "train":
        state["idx"] = torch.arange(case["batch"], dtype=torch.int32, device="cuda")
    return state


# ------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    kind, out = case["kind"], {}
    if kind in ("lattice", "tube"):
        lat = state["lat"]
        lat.step(case["steps"])
        if kind == "tube":
            out["rho"], out["u"], out["own"] = lat.fields()
            out["force"] = lat.force_history()
        else:
            out["rho"], out["ux"], out["uy"], out["own"] = lat.fields(_fields_dtype(case))
            out["force"] = lat.force_history(lat.t - case["steps"], case["steps"])
        return out
    if kind == "batch":
        b = state["batch"]
        b.run(case["steps"], 1e-10, case["steps"] // 2)
        _, _, res, drag = b.status()
        fields = [torch.cat([a.reshape(-1) for a in b.fields(k, _fields_dtype(case))]) for k in range(b.n)]
        return {"residual": np.array(res), "drag": np.array(drag), "fields": torch.cat(fields)}
    net, d = state["net"], state["data"]
    if kind == "train":
        net.train_step(d, state["idx"], 1e-4)
        return {"grads": net.grads()}
    rho, ux, uy = net.infer(d["solid"], d["re"], d["gx"], d["tau"])
    ok = pkg.lbm.warm_check(d["solid"], rho, ux, uy)
    return {"rho": rho, "ux": ux, "uy": uy, "ok": ok}


def _conv_shapes():
    c0, c1, c2, c3 = CH
    return [(2, c0, 0), (c0, c0, 0), (c0, c1, 1), (c1, c1, 1), (c1, c2, 2), (c2, c2, 2), (c2, c3, 3), (c3, c3, 3),
            (2 * c3 + c2, c2, 2), (c2, c2, 2), (c2 + c1, c1, 1), (c1, c1, 1), (c1 + c0, c0, 0), (c0, c0, 0), (c0, 3, 0)]


def work(case):
    kind = case["kind"]
    if kind in ("train", "infer"):
        fwd = [18.0 * ci * co * H * W / 4 ** lv for ci, co, lv in _conv_shapes()]
        params = sum(9 * ci * co + co for ci, co, _ in _conv_shapes())
        if kind == "infer":
            return {"bytes": 4.0 * params + case["batch"] * H * W * 13.0, "flops": case["batch"] * sum(fwd)}
        # forward, weight gradients, input gradients (none of the first layer's)
        return {"bytes": 24.0 * params + case["batch"] * H * W * 13.0, "flops": case["batch"] * (3 * sum(fwd) - fwd[0])}
    if kind == "batch":
        nodes = sum(c["nx"] * c["ny"] for c in lbm_cases.uneven_channels(n_cases=case["cases"]))
        q = 9
    elif kind == "tube":
        nodes, q = case["nx"] * math.pi * (19.34 / 42.0 * case["n"]) ** 2, 19
    else:
        nodes, q = case["nx"] * case["ny"], 9
    # every step takes each fluid node's populations and gives the new ones
    return {"bytes": case["steps"] * nodes * 2.0 * q * BYTES[case["dtype"]],
            "flops": case["steps"] * nodes * (200.0 if q == 9 else 400.0)}


# ------------------------------------------------------------------ in 64 bits
def _d2q9():
    e = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
    return e, [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4


def _d3q19():
    e = [(0, 0, 0)]
    for d in range(3):
        for s in (1, -1):
            e.append(tuple(s if k == d else 0 for k in range(3)))
    for a, b in ((0, 1), (0, 2), (1, 2)):
        for s, t in ((1, 1), (1, -1), (-1, 1), (-1, -1)):
            v = [0, 0, 0]
            v[a], v[b] = s, t
            e.append(tuple(v))
    return e, [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12


WALL = 255


class _Solver:
    """Lattice Boltzmann step with (interpolated) bounce-back, momentum-exchange forces, refill and free bodies, in
    64 bits.  The state is the post-collision one, `post` [q][z][y][x]; two-dimensional lattices have one plane."""

    def __init__(self, dims, shape, tau, g, walls, bodies, device, *, tube=0.0, interpolated=False, mrt=False, refill=0,
                 wall_v=(0.0, 0.0, 0.0)):
        self.two = dims == 2
        e, w = _d2q9() if self.two else _d3q19()
        self.e_list, self.dev = e, device
        self.q = len(e)
        self.e = torch.tensor(e, dtype=torch.float64, device=device)
        self.ei = torch.tensor(e, dtype=torch.int64, device=device)
        self.w = torch.tensor(w, dtype=torch.float64, device=device)
        self.opp = torch.tensor([e.index(tuple(-c for c in v)) for v in e], device=device)
        self.nx, self.ny, self.nz = shape
        self.size = torch.tensor(shape, dtype=torch.int64, device=device)
        self.n = self.nx * self.ny * self.nz
        self.tau, self.walls, self.tube = tau, walls, tube
        self.g = torch.tensor(g, dtype=torch.float64, device=device)
        self.interpolated, self.mrt, self.refill = interpolated, mrt, refill
        self.bodies = bodies  # dicts X, V, Om (lists of 3), r, moves, free (mass, inertia, volume) or None
        self.pressure = None
        self.gravity = (0.0, 0.0, 0.0)
        self.t = 0
        self.x0 = [list(b["X"]) for b in bodies]
        self.duct = None
        if tube > 0.0:
            y = torch.arange(self.ny, device=device).double() - (self.ny - 1) / 2
            z = torch.arange(self.nz, device=device).double() - (self.nz - 1) / 2
            d2 = (y * y)[None, :] + (z * z)[:, None]
            self.duct = (d2 > tube * tube)[:, :, None].expand(self.nz, self.ny, self.nx)
        self.wall_v = wall_v
        self.own = self._raster()
        self.links = self._links()

    # geometry
    def _raster(self):
        own = torch.zeros((self.nz, self.ny, self.nx), dtype=torch.int64, device=self.dev)
        if self.duct is not None:
            own[self.duct] = WALL
        for k, b in enumerate(self.bodies):
            lo = [math.floor(c - b["r"]) - 1 for c in b["X"]]
            hi = [math.ceil(c + b["r"]) + 1 for c in b["X"]]
            if self.two:
                lo[2] = hi[2] = 0
            ax = [torch.arange(lo[d], hi[d] + 1, device=self.dev) for d in range(3)]
            dd = [ax[d].double() - b["X"][d] for d in range(3)]
            d2 = (dd[0] * dd[0])[None, None, :] + (dd[1] * dd[1])[None, :, None]
            if not self.two:
                d2 = d2 + (dd[2] * dd[2])[:, None, None]
            z, y, x = torch.nonzero(d2 <= b["r"] * b["r"], as_tuple=True)
            own[ax[2][z] % self.nz, ax[1][y] % self.ny, ax[0][x] % self.nx] = k + 1
        return own

    def _links(self):
        fluid = self.own == 0
        ns, iss, ss = [], [], []
        for i in range(1, self.q):
            ex, ey, ez = self.e_list[i]
            nb = torch.roll(self.own, (-ez, -ey, -ex), (0, 1, 2))
            if self.walls and ey == 1:
                nb[:, -1, :] = WALL
            elif self.walls and ey == -1:
                nb[:, 0, :] = WALL
            k = torch.nonzero((fluid & (nb != 0)).reshape(-1))[:, 0]
            ns.append(k)
            iss.append(torch.full_like(k, i))
            ss.append(nb.reshape(-1)[k])
        n, i, s = torch.cat(ns), torch.cat(iss), torch.cat(ss)
        return n, i, torch.where(s == WALL, torch.zeros_like(s), s)

    def _coords(self, n):
        return torch.stack([n % self.nx, n // self.nx % self.ny, n // (self.nx * self.ny)], 1)

    def _index(self, c):
        """Flat index of integer coordinates [.., 3] and whether they lie inside the walls."""
        ok = (c[..., 1] >= 0) & (c[..., 1] < self.ny) if self.walls else torch.ones_like(c[..., 0], dtype=torch.bool)
        c = c % self.size
        return (c[..., 2] * self.ny + c[..., 1]) * self.nx + c[..., 0], ok

    def _image(self, d):
        n = self.size.double()
        m = d - n * torch.round(d / n)
        if self.two:
            m = torch.stack([m[:, 0], d[:, 1] if self.walls else m[:, 1], torch.zeros_like(m[:, 0])], 1)
        return m

    def _table(self, key):
        rows = [list(self.wall_v) if key == "V" else [0.0] * 3] + [list(b[key]) for b in self.bodies]
        return torch.tensor(rows, dtype=torch.float64, device=self.dev)

    # collision on [q][m] populations
    def collide(self, f):
        rho = f.sum(0)
        j = torch.stack([sum(c * f[i] for i, v in enumerate(self.e_list) if (c := v[d]) != 0) if not (self.two and d == 2)
                         else torch.zeros_like(rho) for d in range(3)])
        u = j / rho + 0.5 * self.g.reshape(-1, *([1] * (f.dim() - 1)))
        uu = (u * u).sum(0)
        force = [rho * float(self.g[d]) for d in range(3)]
        uf = sum(u[d] * force[d] for d in range(3))
        if self.mrt:
            return self._mrt(f, rho, u, uu, force, uf)
        out = torch.empty_like(f)
        om, pref = 1.0 / self.tau, 1.0 - 0.5 / self.tau
        for i, v in enumerate(self.e_list):
            eu = sum(v[d] * u[d] for d in range(3) if v[d]) + torch.zeros_like(rho)
            ef = sum(v[d] * force[d] for d in range(3) if v[d]) + torch.zeros_like(rho)
            feq = float(self.w[i]) * rho * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * uu)
            out[i] = f[i] - om * (f[i] - feq) + pref * float(self.w[i]) * (3 * (ef - uf) + 9 * eu * ef)
        return out

    def _mrt(self, f, rho, u, uu, force, uf):
        ex, ey = self.e[:, 0], self.e[:, 1]
        e2 = ex * ex + ey * ey
        m = torch.stack([torch.ones_like(ex), 3 * e2 - 4, 4.5 * e2 * e2 - 10.5 * e2 + 4, ex, (3 * e2 - 5) * ex, ey,
                         (3 * e2 - 5) * ey, ex * ex - ey * ey, ex * ey])
        om = 1.0 / self.tau
        s_e, s_p, s_q = lbm.PAPER_MRT_RATES
        s = torch.tensor([0, s_e, s_p, 0, s_q, 0, s_q, om, om], dtype=torch.float64, device=self.dev)
        s = s.reshape(-1, *([1] * (f.dim() - 1)))
        mf = torch.stack([sum(float(m[k, i]) * f[i] for i in range(9)) for k in range(9)])
        ux, uy, fx, fy = u[0], u[1], force[0], force[1]
        meq = torch.stack([rho, -2 * rho + 3 * rho * uu, rho - 3 * rho * uu, rho * ux, -rho * ux, rho * uy, -rho * uy,
                           rho * (ux * ux - uy * uy), rho * ux * uy])
        src = torch.stack([torch.zeros_like(rho), 6 * uf, -6 * uf, fx, -fx, fy, -fy, 2 * (ux * fx - uy * fy),
                           ux * fy + uy * fx])
        # (the conserved rows of mf - meq carry the half-step force; their rates are zero)
        mf = mf - s * (mf - meq) + (1 - 0.5 * s) * src
        inv = torch.linalg.inv(m)
        return torch.stack([sum(float(inv[i, k]) * mf[k] for k in range(9)) for i in range(9)])

    def feq(self, rho, u):
        uu = (u * u).sum(0)
        return torch.stack([float(self.w[i]) * rho * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * uu) for i, v in
                            enumerate(self.e_list) for eu in [sum(v[d] * u[d] for d in range(3))]])

    def start(self, rho, u):
        """f_eq(rho, u), collided once."""
        f = self.feq(rho, u) * (self.own == 0)
        f[:, self.own != 0] = self.w[:, None]
        self.post = self._planes(self.collide(f))

    def _planes(self, post):
        if self.pressure is None:
            return post
        for xb, xf, rb in ((0, 1, self.pressure[0]), (self.nx - 1, self.nx - 2, self.pressure[1])):
            f = post[:, :, :, xf]
            rho = f.sum(0)
            u = torch.einsum("id,izy->dzy", self.e, f) / rho
            uu = (u * u).sum(0)
            eu = torch.einsum("id,dzy->izy", self.e, u)
            new = f + self.w[:, None, None] * (rb - rho) * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * uu)
            ok = (self.own[:, :, xb] == 0) & (self.own[:, :, xf] == 0)
            post[:, :, :, xb] = torch.where(ok, new, post[:, :, :, xb])
        return post

    def _fraction(self, c, e, s):
        """Where the link from c along e meets solid s (0: the duct or a wall)."""
        q = torch.full((len(s),), 0.5, dtype=torch.float64, device=self.dev)
        if not self.interpolated:
            return q
        x, r = self._table("X"), torch.tensor([0.0] + [b["r"] for b in self.bodies], dtype=torch.float64, device=self.dev)
        p = self._image(c.double() - x[s])
        sign = torch.full_like(q, -1.0)
        rad, ee = r[s], e.clone()
        if self.tube > 0.0:
            wall = s == 0
            mid = torch.tensor([0.0, (self.ny - 1) / 2, (self.nz - 1) / 2], dtype=torch.float64, device=self.dev)
            yz = torch.tensor([0.0, 1.0, 1.0], dtype=torch.float64, device=self.dev)
            p = torch.where(wall[:, None], (c.double() - mid) * yz, p)
            ee = torch.where(wall[:, None], ee * yz, ee)
            sign = torch.where(wall, -sign, sign)
            rad = torch.where(wall, torch.full_like(rad, self.tube), rad)
        e2, pe, cc = (ee * ee).sum(1), (p * ee).sum(1), (p * p).sum(1) - rad * rad
        root = (-pe + sign * torch.sqrt(torch.clamp(pe * pe - e2 * cc, min=0.0))) / e2
        root = torch.clamp(torch.where(root <= 0, torch.full_like(root, 1e-12), root), max=1.0)
        return root if self.tube > 0.0 else torch.where(s == 0, q, root)

    def step(self):
        n, i, s = self.links
        flat = self.post.reshape(-1)
        c, e, w = self._coords(n), self.e[i], self.w[i]
        q = self._fraction(c, e, s)
        arm = self._image(c.double() + q[:, None] * e - self._table("X")[s]) * (s > 0)[:, None]
        v = self._table("V")[s] + torch.cross(self._table("Om")[s], arm, dim=1)
        a = flat[i * self.n + n]
        m = 6 * w * (e * v).sum(1)
        back = a - m
        if self.interpolated:
            behind, ok = self._index(c - self.ei[i])
            ok = ok & (self.own.reshape(-1)[behind] == 0)
            near = torch.where(ok, 2 * q * a + (1 - 2 * q) * flat[i * self.n + behind] - m, a - m)
            far = (a - m) / (2 * q) + (1 - 0.5 / q) * flat[self.opp[i] * self.n + n]
            back = torch.where(q < 0.5, near, torch.where(q > 0.5, far, a - m))
        cme = e * (a + back)[:, None]
        gme = (e - v) * a[:, None] + (e + v) * back[:, None]
        rows = torch.cat([cme, torch.cross(arm, cme, dim=1), gme, torch.cross(arm, gme, dim=1)], 1)
        force = torch.zeros((len(self.bodies) + 1, 12), dtype=torch.float64, device=self.dev).index_add_(0, s, rows)
        new = torch.empty_like(self.post)
        for k, (ex, ey, ez) in enumerate(self.e_list):
            new[k] = torch.roll(self.post[k], (ez, ey, ex), (0, 1, 2))
        new.reshape(-1)[self.opp[i] * self.n + n] = back
        self.t += 1
        if any(b["moves"] for b in self.bodies):
            self._move(force, new)
        f = torch.where((self.own == 0)[None], new, self.w.reshape(-1, 1, 1, 1))
        self.post = self._planes(self.collide(f))
        return force[:, [0, 1, 5, 6, 7, 11]] if self.two else force

    def _move(self, force, new):
        rows = force.cpu().numpy()
        for k, b in enumerate(self.bodies):
            if b["free"]:
                mass, inertia, vol = b["free"]
                for d in range(3):
                    b["V"][d] += (rows[k + 1, 6 + d] + (mass - vol) * self.gravity[d]) / mass
                    b["Om"][d] += rows[k + 1, 9 + d] / inertia
                    b["X"][d] += b["V"][d]
            elif b["moves"]:
                b["X"] = [self.x0[k][d] + self.t * b["V"][d] for d in range(3)]
        old, self.own = self.own, self._raster()
        born = torch.nonzero(((old != 0) & (self.own == 0)).reshape(-1))[:, 0]
        if len(born):
            both = ((old == 0) & (self.own == 0)).reshape(-1)
            flat = new.reshape(self.q, -1)
            c = self._coords(born)
            acc = torch.zeros((self.q, len(born)), dtype=torch.float64, device=self.dev)
            count = torch.zeros(len(born), dtype=torch.float64, device=self.dev)
            for k in range(1, self.q):
                at, ok = [], []
                for m in (1, 2, 3):
                    idx, inside = self._index(c + m * self.ei[k])
                    at.append(flat[:, idx])
                    ok.append(inside & both[idx] & (ok[-1] if ok else True))
                a1 = ok[2] if self.refill == 0 else torch.zeros_like(ok[0])
                a2 = ok[1] & ~a1 if self.refill <= 1 else torch.zeros_like(ok[0])
                val = torch.where(a1, 3 * at[0] - 3 * at[1] + at[2], torch.where(a2, 2 * at[0] - at[1], at[0]))
                acc += torch.where(ok[0], val, torch.zeros_like(val))
                count += ok[0].double()
            s = old.reshape(-1)[born]
            arm = self._image(c.double() - self._table("X")[s])
            v = self._table("V")[s] + torch.cross(self._table("Om")[s], arm, dim=1)
            alone = self.feq(torch.ones_like(count), v.T)
            flat[:, born] = torch.where(count > 0, acc / torch.clamp(count, min=1), alone)
        self.links = self._links()

    def fields(self):
        fluid = (self.own == 0).double()
        rho = self.post.sum(0)
        u = torch.stack([sum(v[d] * self.post[i] for i, v in enumerate(self.e_list) if v[d]) / rho if not
                         (self.two and d == 2) else torch.zeros_like(rho) for d in range(3)])
        return rho * fluid, (u - 0.5 * self.g.reshape(3, 1, 1, 1)) * fluid


def _body(X, r, V=(0.0, 0.0, 0.0), moves=False, free=None):
    return {"X": list(X), "r": r, "V": list(V), "Om": [0.0, 0.0, 0.0], "moves": moves, "free": free}


def _plane_solver(lc, device, **kw):
    bodies = [_body((b["cx"], b["cy"], 0.0), b["r"], (b["vx"], b["vy"], 0.0), b["moves"]) for b in lc["bodies"]]
    return _Solver(2, (lc["nx"], lc["ny"], 1), lc["tau"], (lc["gx"], lc["gy"], 0.0), lc["walls_y"], bodies, device,
                   refill=lc["refill"], **kw)


def _rest(s, u0=(0.0, 0.0, 0.0)):
    one = torch.ones((s.nz, s.ny, s.nx), dtype=torch.float64, device=s.dev)
    s.start(one, torch.stack([c * one for c in u0]))


def _poiseuille(s, lc):
    """The steady flow of the channel without its cylinder, half-way walls and their slip included."""
    nu = (lc["tau"] - 0.5) / 3.0
    y = torch.arange(s.ny, dtype=torch.float64, device=s.dev) - 0.5 * (s.ny - 1)
    slip = lc["gx"] * (16.0 * (lc["tau"] - 0.5) ** 2 - 3.0) / (24.0 * nu)
    u = lc["gx"] / (2.0 * nu) * ((0.5 * s.ny) ** 2 - y * y) + slip
    ux = (u - 0.5 * lc["gx"])[None, :, None].expand(s.nz, s.ny, s.nx)
    s.start(torch.ones_like(ux), torch.stack([ux, torch.zeros_like(ux), torch.zeros_like(ux)]))


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "lattice":
        lc, flow = _lattice_inputs(case, seed, device)
        s = _plane_solver(lc, device, interpolated=case["interpolated"], mrt=case["mrt"])
        if case["free"]:
            b = s.bodies[0]
            vol = math.pi * b["r"] ** 2
            b["free"] = (SED_RHO * vol, 0.5 * SED_RHO * vol * b["r"] ** 2, vol)
            s.gravity = (SED_G, 0.0, 0.0)
            _rest(s)
        else:
            rho, ux, uy = (a.double()[None] for a in flow)
            s.start(rho, torch.stack([ux - 0.5 * lc["gx"], uy - 0.5 * lc["gy"], torch.zeros_like(ux)]))
        force = torch.stack([s.step() for _ in range(case["steps"])])
        rho, u = s.fields()
        return {"rho": rho[0], "ux": u[0, 0], "uy": u[1, 0], "own": None, "force": force}
    if kind == "tube":
        tc = _tube_case(case, seed)
        sp = tc["spheres"][0]
        vol = 4.0 / 3.0 * math.pi * sp["r"] ** 3
        free = (TUBE_RHO * vol, 0.4 * TUBE_RHO * vol * sp["r"] ** 2, vol) if case["free"] else None
        s = _Solver(3, (tc["nx"], tc["ny"], tc["nz"]), tc["tau"], tc["g"], False,
                    [_body((sp["cx"], sp["cy"], sp["cz"]), sp["r"], moves=case["free"], free=free)], device,
                    tube=tc["R"], interpolated=case["interpolated"])
        if case["pressure"]:
            s.pressure = (1 + DROP, 1 - DROP)
        _rest(s, tc["u0"])
        force = torch.stack([s.step() for _ in range(case["steps"])])
        rho, u = s.fields()
        return {"rho": rho, "u": u, "own": None, "force": force}
    if kind == "batch":
        fields, drag = [], []
        for lc in _batch_cases(case, seed):
            s = _plane_solver(lc, device)
            _poiseuille(s, lc)
            for _ in range(case["steps"]):
                s.step()
            rho, u = s.fields()
            fields += [rho.reshape(-1), u[0].reshape(-1), u[1].reshape(-1)]
            # the monitor's forces are those of the state it sees, which the next step evaluates
            f = s.step()
            drag.append([float(f[1:, 0].sum()), float(f[1:, 3].sum())])
        return {"residual": None, "drag": np.array(drag), "fields": torch.cat(fields)}
    return _network_exact(case, seed, device)


def _network(layers, x):
    """The warm-start U-Net in 64 bits: 3x3 convolutions as nine shifted matrix products, x periodic, y zero-padded."""

    def conv(x, k, relu=True):
        w, b = layers[k]
        n, h, wd, ci = x.shape
        p = torch.cat([torch.zeros_like(x[:, :1]), x, torch.zeros_like(x[:, :1])], 1)
        p = torch.cat([p[:, :, -1:], p, p[:, :, :1]], 2)
        y = b
        for dy in range(3):
            for dx in range(3):
                y = y + p[:, dy:dy + h, dx:dx + wd].reshape(-1, ci) @ w[:, dy, dx].T
        y = y.reshape(n, h, wd, -1)
        return torch.relu(y) if relu else y

    skips = []
    for lv in range(3):
        x = conv(conv(x, 2 * lv), 2 * lv + 1)
        skips.append(x)
        n, h, w, c = x.shape
        x = x.reshape(n, h // 2, 2, w // 2, 2, c).mean((2, 4))
    x = conv(conv(x, 6), 7)
    mean = x.mean((1, 2), keepdim=True)
    for k, lv in enumerate((2, 1, 0)):
        up = x.repeat_interleave(2, 1).repeat_interleave(2, 2)
        parts = [up, skips[lv]]
        if lv == 2:
            parts.append(mean.expand(-1, up.shape[1], up.shape[2], -1))
        x = conv(conv(torch.cat(parts, 3), 8 + 2 * k), 9 + 2 * k)
    return conv(x, 14, relu=False)


def _network_exact(case, seed, device):
    params, scale = _params(case, seed)
    p = params.double().to(device).requires_grad_(case["kind"] == "train")
    layers, k = [], 0
    for ci, co, _ in _conv_shapes():
        layers.append((p[k:k + co * 9 * ci].reshape(co, 3, 3, ci), p[k + co * 9 * ci:k + co * 9 * ci + co]))
        k += co * 9 * ci + co
    d = _samples(seed, case["batch"], device)
    fluid = (d["solid"] == 0).double()
    x = torch.stack([d["solid"].double(), (d["re"] / 100)[:, None, None].expand_as(fluid)], 3)
    y = _network(layers, x)
    uc = (d["gx"] * H * H / (8 * (d["tau"] - 0.5) / 3))[:, None, None]
    if case["kind"] == "train":
        want = torch.stack([(d["rho"].double() - 1) / (uc * scale), d["ux"].double() / uc, d["uy"].double() / uc], 3)
        loss = (((y - want) ** 2).sum(3) * fluid).sum() / (3 * fluid.sum())
        loss.backward()
        return {"grads": p.grad}
    return {"rho": (1 + uc * scale * y[..., 0]) * fluid, "ux": uc * y[..., 1] * fluid, "uy": uc * y[..., 2] * fluid,
            "ok": None}

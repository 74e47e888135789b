"""The work a user of this library has it do, as timed cases over its public entry points.

Kinds of case:
  run       a domain is advanced several steps and its macroscopic fields are read out
  monitor   a domain is advanced one step at a time, with the mass and momentum after each
            (and the fields after the last)
  strain    steps fused with the strain-rate output (a strain-rate dependent viscosity's loop)
  batch     many uneven channels are advanced together, their residuals checked, their fields read
  obstacles one check of a steady solve: 50 steps of a batch of obstacle channels, the residuals
  train     one training step of the warm-start surrogate (loss, gradients, Adam)
  warm      predicted initial fields for a batch of obstacle channels, written into the solver

`exact` is a plain dense torch implementation in 64 bits of the same model: raw-moment
relaxation matrix, equilibrium in velocity space, streaming by rolls, halfway bounce-back.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2206_00366_amd import rmrt as R
from paper_2206_00366_amd import surrogate as S

WALLS = {"none": 0, "y": R.WALL_YM | R.WALL_YP, "yz": R.WALL_YM | R.WALL_YP | R.WALL_ZM | R.WALL_ZP}
ESIZE = {"f64": 8, "f32dev": 4, "f16dev": 2}
Q = {"Q9": 9, "Q19": 19, "Q27": 27}
FLOPS = {"Q9": 110, "Q19": 300, "Q27": 370}     # of one node update
STRAIN_SPIN_UP = 10                            # steps before a strain case's passes
CHUNK_NODES = 1 << 21                          # nodes the reference collides at a time


def listed():
    return [
        # the smallest domain of the benchmark: a 2D vortex in FP64, launch- and latency-bound
        dict(name="vortex2d_64x32_f64", kind="run", lattice="Q9", eq="NSE", storage="f64", pattern="AB",
             nx=64, ny=32, nz=1, dy=0.5, dz=1.0, walls="none", force=False, steps=100),
        # a live view of a small forced 3D channel: every step is followed by its mass and momentum
        dict(name="monitor3d_48_f32", kind="monitor", lattice="Q19", eq="NSE", storage="f32dev", pattern="AA",
             nx=48, ny=40, nz=36, dy=1.0, dz=1.0, walls="yz", force=True, steps=4),
        # 2D nonlinear convection-diffusion of a hill, the benchmark's grid
        dict(name="hill2d_2048x1024_f32", kind="run", lattice="Q9", eq="NCDE", storage="f32dev", pattern="AA",
             nx=2048, ny=1024, nz=1, dy=0.5, dz=1.0, walls="none", force=False, steps=40),
        # the benchmark's headline: a 3D vortex, FP32 deviation storage
        dict(name="vortex3d_256_f32", kind="run", lattice="Q19", eq="NSE", storage="f32dev", pattern="AA",
             nx=256, ny=256, nz=128, dy=1.0, dz=2.0, walls="none", force=False, steps=20),
        # the same model in half-size storage on an odd grid
        dict(name="vortex3d_odd_f16", kind="run", lattice="Q19", eq="NSE", storage="f16dev", pattern="AA",
             nx=250, ny=203, nz=121, dy=1.0, dz=2.0, walls="none", force=False, steps=20),
        # a reference-accuracy run: FP64 with two buffers
        dict(name="vortex3d_128_f64", kind="run", lattice="Q19", eq="NSE", storage="f64", pattern="AB",
             nx=128, ny=128, nz=96, dy=1.0, dz=2.0, walls="none", force=False, steps=10),
        # a walled, forced 27-velocity channel with the strain rate of every step
        dict(name="strain3d_223x116x100", kind="strain", lattice="Q27", eq="NSE", storage="f32dev", pattern="AA",
             nx=223, ny=116, nz=100, dy=0.5, dz=2.0, walls="yz", force=True, steps=4),
        # uneven 3D channels advanced together (sizes 32..160 per axis)
        dict(name="channels24_32to160", kind="batch", lattice="Q27", storage="f32dev", nd=24, nmin=32, nmax=160,
             steps=20),
        # many small 3D channels (sizes 16..48 per axis)
        dict(name="channels30_16to48", kind="batch", lattice="Q27", storage="f32dev", nd=30, nmin=16, nmax=48,
             steps=20),
        # the inner loop of a steady solve past obstacles
        dict(name="obstacles16_512x256", kind="obstacles", storage="f32dev", nd=16, nx=512, ny=256, steps=50),
        # the warm-start network's training step at its own batch size
        dict(name="train_b16_64x128", kind="train", B=16, H=64, W=128),
        # warm start of a batch of 16 channels with the trained network
        dict(name="warm16_512x256", kind="warm", nd=16, nx=512, ny=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["run", "run", "run", "monitor", "strain", "batch", "obstacles", "train", "warm"])
    if kind in ("run", "monitor", "strain"):
        lattice = rng.choice(["Q9", "Q19", "Q27"])
        storage = rng.choice(["f64", "f32dev", "f32dev", "f16dev"])
        eq = "NCDE" if kind == "run" and lattice == "Q9" and rng.random() < 0.4 else "NSE"
        walls = "none" if eq == "NCDE" else rng.choice(["none", "none", "y" if lattice == "Q9" else "yz"])
        if lattice == "Q9":
            nx, ny, nz = _log_int(rng, 32, 2048), _log_int(rng, 32, 1024), 1
        else:
            hi = {"f64": 144, "f32dev": 192, "f16dev": 208}[storage]
            nx, ny, nz = (_log_int(rng, 24, hi) for _ in range(3))
        if kind == "monitor":
            nx, ny, nz = min(nx, 256), min(ny, 256), min(nz, 64)
        steps = rng.randint(2, 6) if kind != "run" else rng.randint(4, 24)
        return dict(kind=kind, lattice=lattice, eq=eq, storage=storage, pattern=rng.choice(["AA", "AA", "AB"]),
                    nx=nx, ny=ny, nz=nz, dy=rng.choice([0.5, 1.0]), dz=rng.choice([1.0, 2.0]), walls=walls,
                    force=walls != "none" and rng.random() < 0.6, steps=steps)
    if kind == "batch":
        nmin = rng.choice([16, 24, 32])
        return dict(kind="batch", lattice=rng.choice(["Q19", "Q27"]), storage=rng.choice(["f32dev", "f32dev", "f16dev"]),
                    nd=rng.randint(4, 30), nmin=nmin, nmax=rng.randint(nmin + 8, 112), steps=rng.randint(5, 20))
    nx, ny = 4 * _log_int(rng, 32, 128), 4 * _log_int(rng, 16, 64)
    if kind == "obstacles":
        return dict(kind=kind, storage="f32dev", nd=rng.randint(2, 20), nx=nx, ny=ny, steps=50)
    if kind == "warm":
        return dict(kind=kind, nd=rng.randint(2, 20), nx=nx, ny=ny)
    return dict(kind="train", B=rng.randint(2, 16), H=rng.randint(12, 64), W=rng.randint(17, 128))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _single_params(case):
    """The parameter set of a one-domain case, as keyword arguments of make_params."""
    n, dx = (case["nx"], case["ny"], case["nz"]), (1.0, case["dy"], case["dz"])
    p = dict(lattice=case["lattice"], equation=case["eq"], storage=case["storage"], pattern=case["pattern"], n=n, dx=dx,
             wall_faces=WALLS[case["walls"]])
    if case["eq"] == "NCDE":
        p.update(D0=0.01, D2=1.0, adv=(0.05, 0.02, 0.0), rho0=0.0)
    else:
        p.update(nu=0.02 if case["walls"] == "none" else 0.05, nu_b=0.05, rho0=1.0)
        if case["force"]:    # weak enough that no pass of a long run leaves the low-Mach range
            p.update(force=(1e-6, 0.0, 0.0) if case["nz"] == 1 else (1e-6, 0.0, 2.5e-7))
    return p


def _single_fields(case, seed):
    """Initial fields: a Taylor-Green-like vortex with noise of 1e-4 (or a hill), its phases from the seed."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    g = _gen(seed)
    ph = torch.rand(4, generator=g, device="cuda", dtype=torch.float64)
    N = nx * ny * nz
    i = torch.arange(N, device="cuda")
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    if case["eq"] == "NCDE":
        X, Y = x.double(), y.double() * case["dy"]
        Lx, Ly = float(nx), ny * case["dy"]
        s = 0.02 * nx
        dx = torch.remainder(X - ph[0] * Lx + Lx / 2, Lx) - Lx / 2
        dy = torch.remainder(Y - ph[1] * Ly + Ly / 2, Ly) - Ly / 2
        return torch.exp(-(dx * dx + dy * dy) / (2 * s * s)), None
    U0 = 0.02
    X = 2 * math.pi * (x / nx + ph[0])
    Y = 2 * math.pi * (y / ny + ph[1])
    Z = 2 * math.pi * (z / nz + ph[2])
    rho = 1.0 + 1e-4 * (2 * torch.rand(N, generator=g, device="cuda", dtype=torch.float64) - 1)
    if nz == 1:
        u = torch.stack([-U0 * torch.cos(X) * torch.sin(Y), U0 * torch.sin(X) * torch.cos(Y)])
    else:
        u = torch.stack([U0 * torch.sin(X) * torch.cos(Y) * torch.cos(Z), -U0 * torch.cos(X) * torch.sin(Y) * torch.cos(Z),
                         0.1 * U0 * torch.sin(X) * torch.sin(Y)])
    return rho, u


def _channels(case, seed):
    """Parameter sets of uneven force-driven channels: walls on the y and z faces, periodic x.  The sizes are
    the case's own (a program keeps its domains); viscosities and start fields come from the seed."""
    size = random.Random(1000 * case["nd"] + 10 * case["nmin"] + case["nmax"])
    rng = random.Random(seed)
    out = []
    for _ in range(case["nd"]):
        n = tuple(size.randint(case["nmin"], case["nmax"]) for _ in range(3))
        dy, dz = size.choice([0.5, 1.0, 2.0]), size.choice([0.5, 1.0, 2.0])
        nu = rng.uniform(0.01, 0.1)
        H = min(n[1] * dy, n[2] * dz)
        out.append(dict(lattice=case["lattice"], equation="NSE", storage=case["storage"], pattern="AA", n=n,
                        dx=(1.0, dy, dz), nu=nu, nu_b=2 * nu / 3, force=(8 * nu * 0.02 / H**2, 0.0, 0.0), rho0=1.0,
                        wall_faces=WALLS["yz"]))
    return out


def _start_fields(p, k, seed, solid=None):
    """Near-developed start fields of channel k: the parabolic profile across y with 1e-3 relative noise."""
    nx, ny, nz = p["n"]
    N = nx * ny * nz
    g = _gen(seed * 1000 + k)
    y = (torch.arange(N, device="cuda") // nx) % ny
    eta = (y.double() + 0.5) / ny
    d = 2 if nz == 1 else 3
    u = 2e-5 * (2 * torch.rand((d, N), generator=g, device="cuda", dtype=torch.float64) - 1)
    u[0] += 0.02 * 4 * eta * (1 - eta)
    rho = 1.0 + 1e-5 * (2 * torch.rand(N, generator=g, device="cuda", dtype=torch.float64) - 1)
    if solid is not None:
        u[:, solid.reshape(-1).to("cuda") != 0] = 0.0
    return rho, u


def _geometries(case, seed):
    """Obstacle channels: 1-8 circles or rectangles, walls on the y faces, Re 10-100."""
    nx, ny, dy, Ut = case["nx"], case["ny"], 0.5, 0.03
    H = ny * dy
    Y, X = np.meshgrid((np.arange(ny) + 0.5) * dy, np.arange(nx) + 0.5, indexing="ij")
    out = []
    for k in range(case["nd"]):
        rng = random.Random(seed * 1000 + k)
        Re = rng.uniform(10.0, 100.0)
        nu = Ut * H / Re
        solid = np.zeros((ny, nx), dtype=bool)
        for _ in range(rng.randint(1, 8)):
            r = rng.uniform(0.03, 0.09) * H
            cx, cy = rng.uniform(0.12 * nx, 0.88 * nx), rng.uniform(0.07 * H + r, 0.93 * H - r)
            if rng.random() < 0.5:
                solid |= (X - cx) ** 2 + (Y - cy) ** 2 <= r * r
            else:
                solid |= (np.abs(X - cx) <= r) & (np.abs(Y - cy) <= 0.7 * r)
        out.append(dict(solid=solid.reshape(-1), Re=Re, nu=nu, force=(8 * nu * Ut / H**2, 0.0, 0.0), n=(nx, ny, 1),
                        dx=(1.0, dy, 1.0), H=H, Ut=Ut))
    return out


def _net_state(net, seed):
    """The weights, moments and step of a training run under way, from the seed (bf16 weights as the net keeps them)."""
    g = _gen(seed)

    def rnd(t, scale):
        return scale * torch.randn(t.shape, generator=g, device="cuda", dtype=torch.float32)
    for layer in range(4):
        ci = S.CHANS[layer]
        scale = math.sqrt(2.0 / (9 * ci)) * (0.1 if layer == 3 else 1.0)
        net.w32[layer].copy_(rnd(net.w32[layer], scale))
        net.wbf[layer].copy_(net.w32[layer])
        net.b32[layer].copy_(rnd(net.b32[layer], 0.05))
        net.mw[layer].copy_(rnd(net.mw[layer], 1e-3))
        net.mb[layer].copy_(rnd(net.mb[layer], 1e-3))
        net.vw[layer].copy_(1e-5 + rnd(net.vw[layer], 1e-3) ** 2)
        net.vb[layer].copy_(1e-5 + rnd(net.vb[layer], 1e-3) ** 2)
    net.t = 99


def _train_inputs(case, seed):
    g = _gen(seed + 7)
    B, H, W = case["B"], case["H"], case["W"]
    x = torch.zeros((B, H, W, 16), device="cuda")
    x[..., :5] = torch.rand((B, H, W, 5), generator=g, device="cuda")
    T = 0.3 * torch.randn((B, H, W, 3), generator=g, device="cuda")
    Wt = (torch.rand((B, H, W), generator=g, device="cuda") > 0.1).float()
    return x.to(torch.bfloat16), T, Wt


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("run", "monitor", "strain"):
        rho, u = _single_fields(case, seed)
        dom = R.Domain(R.make_params(**_single_params(case)), rho, u)
        if kind == "strain":    # the loop is under way: the stress has left its start value of zero
            dom.step(STRAIN_SPIN_UP)
        return dict(case=case, dom=dom)
    if kind == "batch":
        ps = _channels(case, seed)
        b = R.Batch([R.make_params(**p) for p in ps])
        for k, p in enumerate(ps):
            b.domains[k].set_fields(*_start_fields(p, k, seed))
        b.residuals()     # keeps the velocity that the first check compares with
        return dict(case=case, batch=b)
    if kind == "obstacles":
        geoms = _geometries(case, seed)
        b = S.make_batch(geoms, case["storage"])
        for k, g in enumerate(geoms):
            b.domains[k].set_fields(*_start_fields(g, k, seed, torch.from_numpy(g["solid"])))
        b.residuals()
        return dict(case=case, batch=b)
    if kind == "train":
        net = S.Surrogate(seed=0, B=case["B"], H=case["H"], W=case["W"])
        _net_state(net, seed)
        return dict(case=case, net=net, data=_train_inputs(case, seed))
    geoms = _geometries(case, seed)
    net = S.Surrogate(seed=0, B=case["nd"], H=case["ny"] // S.COARSEN, W=case["nx"] // S.COARSEN)
    _net_state(net, seed)
    return dict(case=case, geoms=geoms, net=net, batch=S.make_batch(geoms))


def _read(d, storage):
    rho, u = d.moments(R.OUT_F64 if storage == "f64" else R.OUT_F32, with_u=d.params.equation == R.NSE)
    return [rho, u]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "run":
        d = state["dom"]
        d.step(case["steps"])
        return _read(d, case["storage"])
    if kind == "monitor":
        d = state["dom"]
        sums = []
        for _ in range(case["steps"]):
            d.step(1)
            sums.append(d.reduce()[:d.d + 1])
        return [np.array(sums)] + _read(d, case["storage"])
    if kind == "strain":
        d = state["dom"]
        dt = R.OUT_F64 if case["storage"] == "f64" else R.OUT_F32
        return [d.step_local(R.GRAD_STRAIN, dt) for _ in range(case["steps"])]
    if kind in ("batch", "obstacles"):
        b = state["batch"]
        b.step(case["steps"])
        r = b.residuals()
        return [np.array(r)] + [_read(d, case["storage"]) for d in b.domains]
    if kind == "train":
        net = state["net"]
        loss = net.loss_and_grads(*state["data"])
        net.adam(1e-3)
        return [loss, list(net.gw), list(net.gb), list(net.w32), list(net.b32)]
    b, net, geoms = state["batch"], state["net"], state["geoms"]
    out, _ = S.predict(net, geoms)
    rho, u = S.initial_fields(geoms, out)
    S.apply_initial(b, rho, u)
    return [out, rho, u, [_read(d, "f32dev") for d in b.domains]]


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------
def _conv_macs(pixels):
    return pixels * 9 * sum(S.CHANS[k] * S.CHANS[k + 1] for k in range(4))


def work(case):
    kind = case["kind"]
    if kind in ("run", "monitor", "strain"):
        N = case["nx"] * case["ny"] * case["nz"]
        d = 2 if case["nz"] == 1 else 3
        es, q = ESIZE[case["storage"]], Q[case["lattice"]]
        o = 8 if case["storage"] == "f64" else 4
        b = 2 * q * es * N
        if kind != "strain":
            b += o * N * (1 if case["eq"] == "NCDE" else 1 + d)
        else:
            b += case["steps"] * o * N * (d * (d + 1) // 2)
        return dict(bytes=b, flops=case["steps"] * N * FLOPS[case["lattice"]])
    if kind == "batch":
        N = sum(p["n"][0] * p["n"][1] * p["n"][2] for p in _channels(case, 0))
        return dict(bytes=N * (2 * Q[case["lattice"]] * ESIZE[case["storage"]] + 3 * 16 + 16),
                    flops=case["steps"] * N * FLOPS[case["lattice"]])
    if kind == "obstacles":
        N = case["nd"] * case["nx"] * case["ny"]
        return dict(bytes=N * (2 * 9 * ESIZE[case["storage"]] + 2 * 16 + 12 + 1), flops=case["steps"] * N * FLOPS["Q9"])
    if kind == "train":
        P = case["B"] * case["H"] * case["W"]
        nw = sum(9 * S.CHANS[k] * S.CHANS[k + 1] + S.CHANS[k + 1] for k in range(4))
        return dict(bytes=P * (16 * 2 + 16) + nw * 4 * 7, flops=6 * _conv_macs(P))
    N = case["nd"] * case["nx"] * case["ny"]
    P = N // S.COARSEN**2
    return dict(bytes=N * (1 + 24 + 36 + 12) + P * 16 * 4, flops=2 * _conv_macs(P) + 150 * N)


# ---------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _velocities(lattice):
    if lattice == "Q9":
        return [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
    e = [(a, b, c) for c in (-1, 0, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)]
    return e if lattice == "Q27" else [v for v in e if abs(v[0]) + abs(v[1]) + abs(v[2]) <= 2]


class _Model:
    """One domain of the rectangular model: dense matrices, (q, N) populations in float64."""

    def __init__(self, p, solid=None):
        self.n, d = p["n"], (2 if p["lattice"] == "Q9" else 3)
        self.d, self.nse, self.rho0 = d, p["equation"] == "NSE", p.get("rho0", 1.0)
        dev = self.dev = "cuda"
        c = np.array(p["dx"][:3], dtype=np.float64)
        if d == 2:
            c[2] = 1.0
        cs2 = self.cs2 = float(min(c[a] ** 2 for a in range(d)) / 3.0)
        self.e = e = np.array(_velocities(p["lattice"]))
        q = len(e)
        self.opp = [int(np.where((e == -e[j]).all(1))[0][0]) for j in range(q)]
        r = cs2 / c**2
        # weights from the moment conditions: sum w = 1, sum w c_a^2 = cs2, sum w c_a^2 c_b^2 = cs2^2
        # (and the tensor-product corner weight on the 27-velocity set)
        w = np.zeros(q)
        if p["lattice"] == "Q19":
            for j in range(q):
                ax = [a for a in range(3) if e[j, a]]
                if len(ax) == 2:
                    w[j] = r[ax[0]] * r[ax[1]] / 4
                elif len(ax) == 1:
                    a = ax[0]
                    w[j] = r[a] / 2 - sum(r[a] * r[b] for b in range(3) if b != a) / 2
            w[[j for j in range(q) if not e[j].any()][0]] = 1 - w.sum()
        else:
            for j in range(q):
                w[j] = np.prod([r[a] / 2 if e[j, a] else 1 - r[a] for a in range(d)])
        C = e * c
        exps = [(a, b, g) for g in range(3 if d == 3 else 1) for b in range(3) for a in range(3)]
        if p["lattice"] == "Q19":
            exps = [x for x in exps if sum(v > 0 for v in x) < 3]
        M = np.array([np.prod(C ** np.array(x), axis=1) for x in exps])
        order = np.array([sum(x) for x in exps])
        sel2 = [exps.index(tuple(2 if a == b else 0 for b in range(3))) for a in range(d)]
        Sm = np.zeros((q, q))
        Minv = np.linalg.inv(M)
        if self.nse:
            nu, nu_b = p["nu"], p.get("nu_b", -1.0)
            nu_b = 2 * nu / d if nu_b < 0 else nu_b
            s_nu = 1 / (0.5 + nu / cs2)
            for k in range(q):
                Sm[k, k] = 1.0 if order[k] <= 1 else s_nu
            g = (c**2 - cs2)[:d]
            ss, sb = 1 / (0.5 + 2 * nu / g), 1 / (0.5 + d * nu_b / g)
            S2 = np.linalg.inv(np.diag(1 / ss) + np.outer((1 / sb - 1 / ss) * g, 1 / g) / d)
            Sm[np.ix_(sel2, sel2)] = S2
            self.IhS = np.eye(3)
            self.IhS[:d, :d] -= S2 / 2
            self.ihs_off = 1 - s_nu / 2
            self.F = np.array(p.get("force", (0.0, 0.0, 0.0)), dtype=np.float64)
            self.nu, self.nu_b = nu, nu_b
            self.S2, self.s_nu = S2, s_nu
        else:
            self.D0, self.D2, self.adv = p["D0"], p["D2"], np.array(p["adv"], dtype=np.float64)
            Sm = np.eye(q)
            P1 = np.diag((order == 1).astype(float))
            self.P1 = torch.tensor(Minv @ P1 @ M, device=dev)
        self.Lam = torch.tensor(Minv @ Sm @ M, device=dev)
        self.c, self.C, self.w, self.q = c, torch.tensor(C, device=dev), w, q
        # rows: 1, c_a / cs2, (c_a^2 - cs2) / (cs2 (C_a^2 - cs2)), c_a c_b / cs2^2
        rows = [np.ones(q)] + [C[:, a] / cs2 for a in range(3)]
        rows += [(C[:, a] ** 2 - cs2) / (cs2 * (c[a] ** 2 - cs2)) if a < d else np.zeros(q) for a in range(3)]
        rows += [C[:, a] * C[:, b] / cs2**2 for a, b in ((0, 1), (0, 2), (1, 2))]
        self.G = torch.tensor((np.array(rows) * w).T.copy(), device=dev)
        nx, ny, nz = self.n
        self.shape = (nz, ny, nx)
        self.solid = None if solid is None else torch.as_tensor(solid, device=dev).bool().reshape(self.shape)
        self.walls = p.get("wall_faces", 0)

    def geq(self, A, B, M2, Mo):
        return self.G @ torch.stack([A, *B, *M2, *Mo])

    def init(self, rho, u):
        f = torch.empty((self.q, rho.numel()), dtype=torch.float64, device=self.dev)
        for s in range(0, rho.numel(), CHUNK_NODES):
            sl = slice(s, s + CHUNK_NODES)
            r = rho[sl]
            if self.nse:
                v = [u[a][sl] if a < self.d else torch.zeros_like(r) for a in range(3)]
                B = [r * v[a] - self.F[a] / 2 for a in range(3)]
            else:
                v = [torch.full_like(r, self.adv[a]) for a in range(3)]
                B = [r * v[a] for a in range(3)]
            f[:, sl] = self.geq(r, B, [r * x * x for x in v], [r * v[0] * v[1], r * v[0] * v[2], r * v[1] * v[2]])
        return f

    def macro(self, f):
        rho = f.sum(0)
        if not self.nse:
            return rho, None
        j = self.C.T @ f
        return rho, torch.stack([(j[a] + self.F[a] / 2) / rho for a in range(3)])

    def collide(self, f):
        rho, u = self.macro(f)
        if not self.nse:
            a = self.adv
            feq = self.geq(rho, [rho * a[k] for k in range(3)], [rho * a[k] ** 2 for k in range(3)],
                           [rho * a[0] * a[1], rho * a[0] * a[2], rho * a[1] * a[2]])
            s1 = 1 / (0.5 + self.D0 * (1 + self.D2 * rho * rho) / self.cs2)
            d = f - feq
            return f - d - (s1 - 1) * (self.P1 @ d)
        F = self.F
        feq = self.geq(rho, [rho * u[a] - F[a] / 2 for a in range(3)], [rho * u[a] ** 2 for a in range(3)],
                       [rho * u[0] * u[1], rho * u[0] * u[2], rho * u[1] * u[2]])
        out = f - self.Lam @ (f - feq)
        if F.any():
            z = torch.zeros_like(rho)
            T = [2 * u[a] * F[a] for a in range(3)]
            Md = [sum(self.IhS[a, b] * T[b] for b in range(self.d)) if a < self.d else z for a in range(3)]
            Mo = [self.ihs_off * (u[a] * F[b] + u[b] * F[a]) for a, b in ((0, 1), (0, 2), (1, 2))]
            out += self.geq(z, [z + F[a] for a in range(3)], Md, Mo)
        return out

    def blocked(self, j):
        """Where the link from a node along e_j meets a wall or a solid node."""
        nz, ny, nx = self.shape
        b = torch.zeros(self.shape, dtype=torch.bool, device=self.dev)
        ex, ey, ez = (int(v) for v in self.e[j])
        w = self.walls
        for ax, v, lo, hi in ((2, ex, 1, 2), (1, ey, 4, 8), (0, ez, 16, 32)):
            idx = [slice(None)] * 3
            if v < 0 and w & lo:
                idx[ax] = 0
                b[tuple(idx)] = True
            if v > 0 and w & hi:
                idx[ax] = self.shape[ax] - 1
                b[tuple(idx)] = True
        if self.solid is not None:
            b |= torch.roll(self.solid, (-ez, -ey, -ex), (0, 1, 2))
        return b

    def step(self, f):
        for s in range(0, f.shape[1], CHUNK_NODES):
            f[:, s:s + CHUNK_NODES] = self.collide(f[:, s:s + CHUNK_NODES])
        new = torch.empty_like(f)
        bounded = self.walls or self.solid is not None
        for j in range(self.q):
            ex, ey, ez = (int(v) for v in self.e[j])
            v = torch.roll(f[j].view(self.shape), (ez, ey, ex), (0, 1, 2))
            if bounded and (ex or ey or ez):
                o = self.opp[j]
                v = torch.where(self.blocked(o), f[o].view(self.shape), v)
            new[j] = v.reshape(-1)
        return new

    def fields(self, f):
        rho, u = self.macro(f)
        if self.solid is not None:
            s = self.solid.reshape(-1)
            rho = torch.where(s, torch.full_like(rho, self.rho0), rho)
            u = torch.where(s, torch.zeros_like(u), u)
        return rho, (None if u is None else u[:self.d])

    def strain(self, f):
        """Strain rate from the second non-equilibrium moments: (xx, yy, [zz,] xy, [xz, yz])."""
        rho, u = self.macro(f)
        d, F = self.d, self.F
        m2 = [[(self.C[:, a] * self.C[:, b]) @ f for b in range(3)] for a in range(3)]
        v = [[m2[a][b] - (rho * self.cs2 if a == b else 0) - rho * u[a] * u[b] + (u[a] * F[b] + F[a] * u[b]) / 2
              for b in range(3)] for a in range(3)]
        tau = {a: -sum(self.IhS[a, b] * v[b][b] for b in range(d)) for a in range(d)}
        K, Kb = rho * self.nu, rho * self.nu_b
        trE = sum(tau.values()) / (d * Kb)
        out = [(tau[a] - (Kb - 2 * K / d) * trE) / (2 * K) for a in range(d)]
        pairs = ((0, 1),) if d == 2 else ((0, 1), (0, 2), (1, 2))
        return torch.stack(out + [-self.ihs_off * v[a][b] / (2 * K) for a, b in pairs])


def _exact_batch(ps, fields, solids, steps):
    res, out = [], []
    for k, p in enumerate(ps):
        m = _Model(p, None if solids is None else solids[k])
        rho, u = fields(k)
        f = m.init(rho, u)
        u0 = m.fields(f)[1]
        for _ in range(steps):
            f = m.step(f)
        r, v = m.fields(f)
        res.append(float(((v - u0).square().sum() / v.square().sum()).sqrt()))
        out.append([r, v])
        del f
    return [np.array(res)] + out


def _silu(y):
    return y / (1 + torch.exp(-y))


def _conv(x, w, b, dil):
    """3x3 dilated convolution of (B, H, W, Cin) with (Cout, 3, 3, Cin), zero outside, tap by tap."""
    B, H, W, _ = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, dil, dil, dil, dil))
    y = torch.zeros((B * H * W, w.shape[0]), dtype=torch.float64, device=x.device)
    for ky in range(3):
        for kx in range(3):
            y += xp[:, ky * dil:ky * dil + H, kx * dil:kx * dil + W].reshape(B * H * W, -1) @ w[:, ky, kx].T.contiguous()
    return (y + b).view(B, H, W, -1)


def _net64(net, x):
    w = [t.double().requires_grad_() for t in net.wbf]
    b = [t.double().requires_grad_() for t in net.b32]
    a = x.double()
    for layer in range(4):
        a = _conv(a, w[layer], b[layer], S.DILS[layer])
        if layer < 3:
            a = _silu(a)
    return a, w, b


def exact(case, seed):
    kind = case["kind"]
    if kind in ("run", "monitor", "strain"):
        m = _Model(_single_params(case))
        f = m.init(*_single_fields(case, seed))
        sums, strains = [], []
        for _ in range(STRAIN_SPIN_UP if kind == "strain" else 0):
            f = m.step(f)
        for _ in range(case["steps"]):
            if kind == "strain":
                strains.append(m.strain(f))
            f = m.step(f)
            if kind == "monitor":
                rho, u = m.macro(f)
                sums.append([float(rho.sum())] + [float((rho * u[a]).sum()) for a in range(m.d)])
        if kind == "strain":
            return strains
        return ([np.array(sums)] if kind == "monitor" else []) + list(m.fields(f))
    if kind == "batch":
        ps = _channels(case, seed)
        return _exact_batch(ps, lambda k: _start_fields(ps[k], k, seed), None, case["steps"])
    if kind == "obstacles":
        gs = _geometries(case, seed)
        ps = [dict(lattice="Q9", equation="NSE", n=g["n"], dx=g["dx"], nu=g["nu"], force=g["force"], rho0=1.0,
                   wall_faces=WALLS["y"]) for g in gs]
        return _exact_batch(ps, lambda k: _start_fields(gs[k], k, seed, torch.from_numpy(gs[k]["solid"])),
                            [g["solid"] for g in gs], case["steps"])
    if kind == "train":
        net = S.Surrogate(seed=0, B=case["B"], H=case["H"], W=case["W"])
        _net_state(net, seed)
        x, T, Wt = _train_inputs(case, seed)
        y, w, b = _net64(net, x)
        loss = (Wt.double()[..., None] * (y[..., :3] - T.double()) ** 2).sum() / Wt.double().sum()
        loss.backward()
        new = []
        for t, g, mo, vo in ([(net.w32[k], w[k].grad, net.mw[k], net.vw[k]) for k in range(4)]
                             + [(net.b32[k], b[k].grad, net.mb[k], net.vb[k]) for k in range(4)]):
            mm = 0.9 * mo.double() + 0.1 * g
            vv = 0.999 * vo.double() + 0.001 * g * g
            new.append(t.double() - 1e-3 * (mm / (1 - 0.9**100)) / ((vv / (1 - 0.999**100)).sqrt() + 1e-8))
        return [float(loss), [t.grad for t in w], [t.grad for t in b], new[:4], new[4:]]
    gs = _geometries(case, seed)
    nx, ny, k, nd = case["nx"], case["ny"], S.COARSEN, case["nd"]
    H, W, dy, Ut = ny // k, nx // k, 0.5, 0.03
    net = S.Surrogate(seed=0, B=nd, H=H, W=W)
    _net_state(net, seed)
    solid = torch.tensor(np.stack([g["solid"].reshape(ny, nx) for g in gs]), device="cuda")
    sf = solid.double()
    x = torch.zeros((nd, H, W, 16), dtype=torch.float64, device="cuda")
    x[..., 0] = sf.view(nd, H, k, W, k).mean((2, 4))
    yc = (torch.arange(H, device="cuda").double() * k + 0.5 * k) * dy
    x[..., 1] = (4 * yc * (ny * dy - yc) / (ny * dy) ** 2)[None, :, None]
    x[..., 2] = torch.tensor([g["Re"] / S.RE_SCALE for g in gs], device="cuda", dtype=torch.float64)[:, None, None]
    x[..., 3] = sf.mean(1).view(nd, 1, W, k).mean(3)
    x[..., 4] = sf.mean((1, 2))[:, None, None]
    with torch.no_grad():
        out = _net64(net, x)[0]

    def lerp(n, m):
        p = ((torch.arange(n, device="cuda").double() + 0.5) / k - 0.5).clamp(0, m - 1)
        i0 = p.floor().long()
        return i0, (i0 + 1).clamp(max=m - 1), p - i0
    y0, y1, fy = lerp(ny, H)
    x0, x1, fx = lerp(nx, W)
    o = out[..., :3]
    fx, fy = fx[None, None, :, None], fy[None, :, None, None]
    o = ((o[:, y0][:, :, x0] * (1 - fx) + o[:, y0][:, :, x1] * fx) * (1 - fy)
         + (o[:, y1][:, :, x0] * (1 - fx) + o[:, y1][:, :, x1] * fx) * fy)
    yf = (torch.arange(ny, device="cuda").double() + 0.5) * dy
    prior = (4 * yf * (ny * dy - yf) / (ny * dy) ** 2)[None, :, None]
    rho = 1 + o[..., 2] / S.RHO_SCALE
    u = torch.stack([Ut * (prior + o[..., 0]), Ut * o[..., 1]], 1)
    u = torch.where(solid[:, None], torch.zeros_like(u), u)
    reads = []
    for i in range(nd):
        s = solid[i]
        reads.append([torch.where(s, torch.ones_like(rho[i]), rho[i]).reshape(-1),
                      torch.where(s, torch.zeros_like(u[i]), u[i]).reshape(2, -1)])
    return [out, rho.reshape(nd, -1), u.reshape(nd, 2, -1), reads]

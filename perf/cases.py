"""The work that programs have this library do, as cases that can be timed and checked.

A program holds a `sim.GpuSim`, `sim.OpenSim` or `sim.Ensemble` and steps it (the "step", "open" and "ensemble" cases), or calls the
entry points of `hvpic` itself on stores of its own (the "particles", "fields" and "start" cases), or trains and applies the field
surrogate (the "train" and "predict" cases).  Inputs are drawn on the GPU from the seed, with the densities, temperatures, drifts and
time steps of the repository's workloads.

What comes back: the fields, the moments and, where the order of the store is settled by the case's own integers, the whole store with
its map and cell_start.  The FP64 diagnostics are computed as by default but not returned: they are sums of FP32 partials, and their
type promises more digits than they carry.  `exact` gives no value for offsets and cells: an ion within rounding of a face may be kept
from either side of it.
"""
import math

import numpy as np
import torch

from paper_2305_05600_amd import hvpic as H
from paper_2305_05600_amd import sim as S
from paper_2305_05600_amd import workloads as W

DEV = "cuda"
STORE = ("cell", "ox", "oy", "oz", "ux", "uy", "uz", "w")


# ------------------------------------------------------------------ the list

def _step(name=None, **kw):
    c = dict(kind="step", flavour="alfven", nx=32, ny=32, nz=1, ppc=64.0, nsub=4, shape="qs", gather_map=True, energy_eq=False, smooth=0)
    c.update(kw)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # the smallest run in use (the periodic test box): every launch and host call shows
        _step("step_small", nx=32, ny=32, ppc=64.0),
        # the benchmark's double Harris sheet, whole steps in its sequence
        _step("step_harris", flavour="harris", nx=512, ny=256, ppc=100.0, nsub=10),
        # GpuSim as its defaults make it (the store moved by the sort): few ions per cell, an odd grid, smoothed moments and fields
        _step("step_default_sparse", nx=413, ny=257, ppc=36.0, gather_map=False, smooth=2),
        # a run with the electron energy equation, heat conduction and hyper-resistivity
        _step("step_energy_eq", nx=256, ny=192, ppc=64.0, energy_eq=True),
        # the 3D core + beam box at an eighth of its full size, whole steps
        _step("step_beam3d", flavour="beam", nx=64, ny=64, nz=64, ppc=64.0),
        # the solar-wind box open in x, at half its full size along each axis
        dict(name="open_wind", kind="open", nx=400, ny=800, ppc=100, nsub=5, shape="ngp"),
        # independent runs of uneven size stepped together, replayed from a graph
        dict(name="ensemble_8", kind="ensemble", runs=8, side_lo=64, side_hi=256, ppc_lo=32, ppc_hi=200, pick=4),
        # the largest store in use: push through the map and the sort of the full 3D beam box
        dict(name="particles_3d_full", kind="particles", nx=128, ny=128, nz=128, ppc=64.0, shape="qs"),
        # the field advance of that box on its own
        dict(name="fields_3d_full", kind="fields", nx=128, ny=128, nz=128, nsub=4),
        # what starts or restarts a run: the general sort of an unsorted store, its moments and E
        dict(name="start_harris", kind="start", nx=512, ny=256, nz=1, ppc=100.0, shape="qs"),
        # the surrogate proposing one field advance of the Harris grid
        dict(name="surrogate_predict", kind="predict", nx=512, ny=256),
        # one training step of it at the benchmark's batch
        dict(name="surrogate_train", kind="train", nx=512, ny=256, batch=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step2d"] * 5 + ["harris", "step3d", "step3d", "open", "open", "ensemble", "particles", "particles", "fields",
                                        "start", "predict", "train"])
    shape = rng.choice(["qs", "qs", "ngp"])
    if kind == "step2d":
        nx, ny = _log(rng, 24, 512), _log(rng, 24, 512)
        eq = rng.random() < 0.25
        return _step(nx=nx, ny=ny, ppc=round(rng.uniform(24.0, min(200.0, 1.3e7 / (nx * ny))), 1), nsub=rng.randint(2, 10), shape=shape,
                     gather_map=rng.random() < 0.6, energy_eq=eq, smooth=0 if eq else rng.choice([0, 0, 0, 1, 2]))
    if kind == "harris":
        return _step(flavour="harris", nx=rng.randint(192, 512), ny=rng.randint(128, 256), ppc=round(rng.uniform(60.0, 100.0), 1), nsub=10)
    if kind == "step3d":
        nx, ny, nz = (_log(rng, 12, 72) for _ in range(3))
        return _step(flavour="beam", nx=nx, ny=ny, nz=nz, ppc=round(rng.uniform(24.0, 64.0), 1), shape=shape, gather_map=rng.random() < 0.7)
    if kind == "open":
        return dict(kind="open", nx=_log(rng, 48, 500), ny=_log(rng, 48, 800), ppc=rng.randint(30, 100), nsub=rng.randint(2, 6), shape=shape)
    if kind == "ensemble":
        return dict(kind="ensemble", runs=rng.randint(3, 10), side_lo=64, side_hi=rng.choice([128, 192, 256]), ppc_lo=32,
                    ppc_hi=rng.choice([64, 128, 200]), pick=rng.randint(1, 1 << 20))
    if kind == "particles":
        if rng.random() < 0.5:
            nx, ny, nz = _log(rng, 40, 600), _log(rng, 40, 600), 1
        else:
            nx, ny, nz = (_log(rng, 14, 110) for _ in range(3))
        return dict(kind="particles", nx=nx, ny=ny, nz=nz, ppc=round(rng.uniform(24.0, 64.0 if nz > 1 else 120.0), 1), shape=shape)
    if kind == "fields":
        nz = rng.choice([1, _log(rng, 12, 128)])
        return dict(kind="fields", nx=_log(rng, 12, 128) * (4 if nz == 1 else 1) + rng.randint(0, 3), ny=_log(rng, 12, 128), nz=nz,
                    nsub=rng.randint(2, 10))
    if kind == "start":
        return dict(kind="start", nx=_log(rng, 40, 512), ny=_log(rng, 40, 256), nz=1, ppc=round(rng.uniform(24.0, 100.0), 1), shape=shape)
    nx, ny = _log(rng, 60, 512), _log(rng, 60, 256)
    return dict(kind="predict", nx=nx, ny=ny) if kind == "predict" else dict(kind="train", nx=nx, ny=ny, batch=rng.randint(2, 8))


# -------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uni(g, n, lo=0.0, hi=1.0):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * (hi - lo) + lo


def _offset(x64):
    """FP32 offsets in [-1, 1)."""
    return x64.float().clamp(-1.0, float(np.nextafter(np.float32(1.0), np.float32(0.0))))


def _config(c):
    """The run parameters of a case (the repository's workloads' values)."""
    kind, shape = c["kind"], W.SHAPE_QS if c.get("shape", "qs") == "qs" else W.SHAPE_NGP
    nx, ny, nz = c["nx"], c["ny"], c.get("nz", 1)
    base = dict(name="case", ndim=3 if nz > 1 else 2, nx=nx, ny=ny, nz=nz, shape=shape, nsub=c.get("nsub", 4))
    if kind == "open":
        base["nx"] = nx + 2
        return W.Config(**base, dx=2.0, dy=2.0, dz=1.0, dt=0.002, te=0.25, eta=1e-3, open_x=1, buffer_cells=8, eta_h_buffer=1.0)
    if nz > 1:
        return W.Config(**base, dx=1.0, dy=1.0, dz=1.0, dt=0.05, te=1.0, eta=1e-4)
    if c.get("flavour") == "harris" or kind in ("start", "predict", "train"):
        return W.Config(**base, dx=0.125, dy=0.125, dz=1.0, dt=0.003, te=0.5 / 6.0, eta=1e-3)
    extra = dict(gamma_e=5.0 / 3.0, energy_eq=1, kappa0=0.05, eta_h=1e-3) if c.get("energy_eq") else {}
    return W.Config(**base, dx=0.5, dy=0.5, dz=1.0, dt=0.01, te=0.25, eta=1e-3, nsmooth=c.get("smooth", 0), **extra)


def _centres(cfg):
    c = torch.arange(cfg.ncell, device=DEV)
    return ((c % cfg.nx) + 0.5) * cfg.dx, (((c // cfg.nx) % cfg.ny) + 0.5) * cfg.dy, ((c // (cfg.nx * cfg.ny)) + 0.5) * cfg.dz


def _ions(cfg, flavour, ppc, g):
    """An unsorted store: cell, offsets, velocities, weight (GPU tensors)."""
    n = int(round(ppc * cfg.ncell))
    V = cfg.dx * cfg.dy * cfg.dz
    if flavour == "harris":
        L, ti = 0.5, 0.5 / 1.2
        Lx, Ly = cfg.nx * cfg.dx, cfg.ny * cfg.dy
        sheet, back = 2.0 * L * Lx, 0.2 * Lx * Ly
        ns = int(round(n * sheet / (2 * sheet + back)))
        u = _uni(g, 2 * ns).clamp(1e-12, 1 - 1e-12)
        y0 = torch.cat([torch.full((ns,), 0.25 * Ly, device=DEV, dtype=torch.float64), torch.full((ns,), 0.75 * Ly, device=DEV, dtype=torch.float64)])
        y = torch.cat([_uni(g, n - 2 * ns, 0.0, Ly), y0 + L * torch.atanh(2.0 * u - 1.0)])
        vel = torch.randn((3, n), generator=g, device=DEV) * math.sqrt(ti)
        vel[2, n - 2 * ns:n - ns] -= 2.0 * ti / L
        vel[2, n - ns:] += 2.0 * ti / L
        order = torch.randperm(n, generator=g, device=DEV)
        sx, sy = _uni(g, n, 0.0, cfg.nx), torch.remainder(y[order], Ly) / cfg.dy
        i, j = sx.floor().clamp(0, cfg.nx - 1), sy.floor().clamp(0, cfg.ny - 1)
        p = dict(cell=(i + cfg.nx * j).int(), ox=_offset(2 * (sx - i) - 1), oy=_offset(2 * (sy - j) - 1))
        p.update(ux=vel[0][order].contiguous(), uy=vel[1][order].contiguous(), uz=vel[2][order].contiguous())
        p["w"] = torch.full((n,), (2 * sheet + back) / n, device=DEV)
        return p
    if flavour == "wind":
        col = torch.randint(0, (cfg.nx - 2) * cfg.ny, (n,), generator=g, device=DEV)
        cell = (col % (cfg.nx - 2) + 1 + cfg.nx * (col // (cfg.nx - 2))).int()
    else:
        cell = torch.randint(0, cfg.ncell, (n,), generator=g, device=DEV, dtype=torch.int32)
    p = dict(cell=cell, ox=_offset(_uni(g, n, -1.0, 1.0)), oy=_offset(_uni(g, n, -1.0, 1.0)))
    if cfg.ndim == 3:
        p["oz"] = _offset(_uni(g, n, -1.0, 1.0))
    vth = 1.0 if flavour == "beam" else 0.5
    for a in "xyz":
        p["u" + a] = torch.randn(n, generator=g, device=DEV) * vth
    p["w"] = torch.full((n,), V / ppc, device=DEV)
    if flavour == "beam":  # an eighth of the ions carry a twentieth of the density at 10 v_A, without net current
        beam = torch.rand(n, generator=g, device=DEV) < 0.125
        p["ux"] += torch.where(beam, 10.0, -0.05 * 10.0 / 0.95)
        p["w"] = torch.where(beam, 0.05 / 0.125, 0.95 / 0.875) * (V / ppc)
    if flavour == "wind":
        p["ux"] += 10.0
    return p


def _field(cfg, flavour, amp=0.01):
    x, y, _ = _centres(cfg)
    B = torch.zeros((3, cfg.ncell), device=DEV, dtype=torch.float64)
    if flavour == "harris":
        L, Lx, Ly = 0.5, cfg.nx * cfg.dx, cfg.ny * cfg.dy
        kx, ky = 2 * math.pi / Lx, 2 * math.pi / Ly
        dbx, dby = -ky * torch.cos(kx * x) * torch.cos(ky * y), -kx * torch.sin(kx * x) * torch.sin(ky * y)
        s = 0.05 / float((dbx * dbx + dby * dby).max().sqrt())
        B[0] = torch.tanh((y - 0.25 * Ly) / L) - torch.tanh((y - 0.75 * Ly) / L) - 1.0 + s * dbx
        B[1] = s * dby
    elif flavour == "wind":
        B[2] = 0.05 * torch.sin(2 * math.pi * x / (cfg.nx * cfg.dx))
    else:
        B[0] = 1.0
        if flavour == "alfven":
            B[1] = amp * torch.cos(2 * math.pi * x / (cfg.nx * cfg.dx))
    return B.float()


def _waves(cfg, g, ncomp, amp, noise):
    """ncomp smooth arrays (a few long modes) of the given amplitude with grid-scale noise."""
    xyz = _centres(cfg)
    ext = (cfg.nx * cfg.dx, cfg.ny * cfg.dy, cfg.nz * cfg.dz)
    out = torch.zeros((ncomp, cfg.ncell), device=DEV, dtype=torch.float64)
    for a in range(ncomp):
        for _ in range(3):
            r = _uni(g, 4).tolist()
            ph = sum(2 * math.pi * (1 + int(2 * r[q])) * xyz[q] / ext[q] for q in range(cfg.ndim)) + 6.28 * r[3]
            out[a] += amp / 3 * torch.cos(ph)
        out[a] += noise * torch.randn(cfg.ncell, generator=g, device=DEV, dtype=torch.float64)
    return out


def _numpy(parts):
    return {k: v.cpu().numpy() for k, v in parts.items()}


def _store(parts, ndim):
    n = parts["cell"].numel()
    p = H.Particles(ndim, max(n, 1), DEV)
    p.n = n
    for k in STORE:
        if getattr(p, k) is not None:
            getattr(p, k)[:n].copy_(parts[k])
    return p


def _arrays(p, n=None):
    n = p.n if n is None else n
    return {k: getattr(p, k)[:n] for k in STORE if getattr(p, k) is not None}


def _ens_specs(c, seed):
    """The runs' sizes are the case's, their contents the seed's."""
    r = np.random.Generator(np.random.PCG64(c["pick"]))
    q = np.random.Generator(np.random.PCG64(seed))
    return [dict(side=int(r.integers(c["side_lo"], c["side_hi"] + 1)), ppc=float(r.integers(c["ppc_lo"], c["ppc_hi"] + 1)),
                 te=float(0.25 * q.uniform(0.1, 1.0)), amp=float(q.uniform(0.001, 0.05))) for _ in range(c["runs"])]


def _ens_run(sp, g):
    cfg = _config(dict(kind="step", nx=sp["side"], ny=sp["side"])).replace(te=sp["te"])
    return cfg, _ions(cfg, "alfven", sp["ppc"], g), _field(cfg, "alfven", sp["amp"])


def _moved(cfg, c, g):
    """A store in the order of the cells its ions held one step ago, the map that sorts it, and cell_start: what a step finds."""
    p = _ions(cfg, "beam" if cfg.ndim == 3 else "alfven", c["ppc"], g)
    n = cfg.nx, cfg.ny, cfg.nz
    cell = p["cell"].long()
    idx = [cell % n[0], (cell // n[0]) % n[1], cell // (n[0] * n[1])]
    h = (cfg.dx, cfg.dy, cfg.dz)
    for a, (o, u) in enumerate((("ox", "ux"), ("oy", "uy"), ("oz", "uz"))[:cfg.ndim]):
        back = p[o] - p[u] * (2.0 * cfg.dt / h[a])
        idx[a] = torch.remainder(idx[a] + (back >= 1.0).long() - (back < -1.0).long(), n[a])
    order = torch.argsort((idx[0] + n[0] * (idx[1] + n[1] * idx[2])).int(), stable=True)
    p = {k: v[order].contiguous() for k, v in p.items()}
    perm = torch.argsort(p["cell"], stable=True).int()
    cs = torch.zeros(cfg.ncell + 1, dtype=torch.int32, device=DEV)
    cs[1:] = torch.bincount(p["cell"].long(), minlength=cfg.ncell).cumsum(0).int()
    return p, perm, cs


def _eb(cfg, g):
    """E and B as a push of such a box finds them."""
    B = _waves(cfg, g, 3, 0.05, 0.01)
    B[0] += 1.0
    return _waves(cfg, g, 3, 0.1, 0.05).float(), B.float()


def _moments(cfg, g):
    n, nprev = 1.0 + _waves(cfg, g, 1, 0.05, 1e-3)[0], 1.0 + _waves(cfg, g, 1, 0.05, 1e-3)[0]
    return n.float(), _waves(cfg, g, 3, 0.02, 1e-3).float(), nprev.float(), _waves(cfg, g, 3, 0.02, 1e-3).float()


TRAIN_LR, TRAIN_WARM = 1e-3, 3


def _net(c, seed, g):
    """Weights of a network under training, the normalisation and snapshots of the field advance."""
    cfg = _config(c)
    r = np.random.Generator(np.random.PCG64(seed))
    wts = [(w, r.uniform(-0.2, 0.2, b.size)) for w, b in S.Surrogate.initial_weights(int(r.integers(1 << 30)))]
    norm = (np.array([0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0]), np.array([0.6, 0.05, 0.05, 0.3, 0.1, 0.1, 0.3]), np.array([2e-3, 2e-3, 2e-3]))
    k = 2 * c["batch"] if c["kind"] == "train" else 1
    P = cfg.ncell
    data = [torch.empty((k, 3, P), device=DEV), torch.empty((k, P), device=DEV), torch.empty((k, 3, P), device=DEV), torch.empty((k, 3, P), device=DEV)]
    base = _field(cfg, "harris").double()
    for s in range(k):
        B = base + _waves(cfg, g, 3, 0.03, 5e-3)
        J = _waves(cfg, g, 3, 0.1, 0.02)
        data[0][s], data[1][s], data[2][s] = B, 1.0 + _waves(cfg, g, 1, 0.3, 0.03)[0], J
        data[3][s] = B + 2e-3 * torch.tanh(3 * J) + 1e-3 * (torch.roll(B, 1, -1) - B)
    idx = torch.from_numpy(np.stack([r.choice(k, c.get("batch", 1), replace=False) for _ in range(TRAIN_WARM + 1)]).astype(np.int32)).to(DEV)
    return cfg, wts, norm, data, idx


# -------------------------------------------------------------- prepare, run

# what the autotuner settles on for the benchmark's ensemble (the steps it tunes on would leave another state each time)
TUNED = dict(push_chunk=[1, 2, 2], field_tile=[0, 1], blocks_per_cu=[4, 2, 8, 2])
INFLOW = dict(n=1.0, ux=10.0, uy=0.0, uz=0.0, vth=0.5, faces=3)


def prepare(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind == "ensemble":
        runs = [_ens_run(sp, g) for sp in _ens_specs(c, seed)]
        sims = [S.GpuSim(cfg, _numpy(p), B.cpu().numpy(), gather_map=True) for cfg, p, B in runs]
        ens = S.Ensemble(sims)
        ens.set_tuning(TUNED)
        ens.capture(True)
        return dict(kind=kind, ens=ens, sims=sims, mom=[((s.n_prev, s.J_prev), (s.n_half, s.J_half)) for s in sims])
    cfg = _config(c)
    if kind == "step":
        p, B = _ions(cfg, c["flavour"], c["ppc"], g), _field(cfg, c["flavour"])
        return dict(kind=kind, sim=S.GpuSim(cfg, _numpy(p), B.cpu().numpy(), gather_map=c["gather_map"]))
    if kind == "open":
        p, B1 = _ions(cfg, "wind", c["ppc"] * (cfg.nx - 2) / cfg.nx, g), _field(cfg, "wind")
        p["w"].fill_(cfg.dx * cfg.dy * cfg.dz / c["ppc"])
        B0 = np.zeros((3, cfg.ncell), np.float32)
        B0[1] = 1.0
        return dict(kind=kind, sim=S.OpenSim(cfg, _numpy(p), B0, B1.cpu().numpy(), dict(INFLOW, ppc=c["ppc"]), seed=seed))
    f32 = dict(dtype=torch.float32, device=DEV)
    s = dict(kind=kind, cfg=cfg)
    nc = cfg.ncell
    if kind == "particles":
        p, perm, cs = _moved(cfg, c, g)
        s["E"], s["B"] = _eb(cfg, g)
        s["p"], s["perm"], s["cs"] = _store(p, cfg.ndim), perm, cs
        del p
        s["q"] = H.Particles(cfg.ndim, perm.numel(), DEV)
        s["perm2"], s["cs2"] = torch.empty_like(perm), torch.empty_like(cs)
        s["n"], s["J"] = torch.empty(nc, **f32), torch.empty((3, nc), **f32)
        s["diag"] = torch.zeros(4, dtype=torch.float64, device=DEV)
        s["ctx"] = H.Context(cfg, perm.numel(), DEV)
    elif kind == "start":
        p = _ions(cfg, "harris", c["ppc"], g)
        s["p"], s["q"] = _store(p, 2), H.Particles(2, p["cell"].numel(), DEV)
        s["B"], s["E"] = _field(cfg, "harris"), torch.empty((3, nc), **f32)
        s["cs"] = torch.empty(nc + 1, dtype=torch.int32, device=DEV)
        s["n"], s["J"] = torch.empty(nc, **f32), torch.empty((3, nc), **f32)
        s["ctx"] = H.Context(cfg, s["p"].n, DEV)
    elif kind == "fields":
        _, s["B"] = _eb(cfg, g)
        s["mom"] = _moments(cfg, g)
        s["E"] = torch.empty((3, nc), **f32)
        s["diag"] = torch.zeros(3, dtype=torch.float64, device=DEV)
        s["ctx"] = H.Context(cfg, 1, DEV)
    else:
        cfg, wts, norm, data, idx = _net(c, seed, g)
        net = S.Surrogate(cfg.nx, cfg.ny, batch=c.get("batch", 1))
        net.load(wts, norm)
        s.update(net=net, data=data, idx=idx)
        if kind == "train":
            s["loss"] = torch.zeros(1, dtype=torch.float64, device=DEV)
            s["w"] = torch.empty(sum(o * 9 * i for i, o in net.LAYERS), **f32)
            s["b"] = torch.empty(sum(o for _, o in net.LAYERS), **f32)
            for k in range(TRAIN_WARM):  # the moments of Adam fill at rate 0, as under a warm-up
                _train_step(s, k, 0.0)
        else:
            s["in"] = tuple(t[0].contiguous() for t in data[:3])
    return s


def _train_step(s, k, lr):
    B, n, J, Bt = s["data"]
    net = s["net"]
    H.hvpic_no_train_step(net.params, net.ws_train, net.nx, net.ny, B, n, J, Bt, s["idx"][k], lr, s["loss"])


def run(s):
    kind = s["kind"]
    if kind == "step":
        m = s["sim"]
        m.step()
        out = dict(E=m.E, B=m.B, n=m.n_prev, J=m.J_prev, cell_start=m.cs, store=_arrays(m.p))
        if m.gather_map:
            out["map"] = m.perm
        if m.pe is not None:
            out["pe"] = m.pe
        return out
    if kind == "open":
        m = s["sim"]
        m.step()
        # (the store's length is the step's own: how many ions came and went)
        return dict(E=m.E, B1=m.B1, B=m.Btot, n=m.n_prev, J=m.J_prev, cell_start=m.cs[:m.cfg.ncell + 1])
    if kind == "ensemble":
        e = s["ens"]
        e.step()
        k = e.steps & 1
        return [dict(E=m.E, B=m.B, n=q[k][0], J=q[k][1]) for m, q in zip(s["sims"], s["mom"])]
    if kind == "particles":
        c = s["ctx"].ctx
        H.hvpic_gather_push_perm(c, s["p"], s["perm"], s["q"], s["cs"], s["E"], s["B"], s["n"], s["J"], s["diag"])
        H.hvpic_sort_perm(c, s["q"], s["cs"], s["perm2"], s["cs2"])
        return dict(store=_arrays(s["q"]), n=s["n"], J=s["J"], map=s["perm2"], cell_start=s["cs2"])
    if kind == "start":
        c = s["ctx"].ctx
        H.hvpic_sort(c, s["p"], s["q"], None, s["cs"], full=True)
        H.hvpic_deposit(c, s["q"], s["cs"], 0.0, s["n"], s["J"])
        H.hvpic_field_advance(c, s["B"], s["n"], s["J"], None, None, s["E"], mode=1)
        return dict(store=_arrays(s["q"]), cell_start=s["cs"], n=s["n"], J=s["J"], E=s["E"])
    if kind == "fields":
        n, J, npv, Jp = s["mom"]
        H.hvpic_field_advance(s["ctx"].ctx, s["B"], n, J, npv, Jp, s["E"], mode=0, diag_out=s["diag"])
        return dict(B=s["B"], E=s["E"])
    if kind == "predict":
        return s["net"].predict(*s["in"])
    _train_step(s, TRAIN_WARM, TRAIN_LR)
    H.hvpic_no_store(s["net"].params, s["w"], s["b"])
    return dict(w=s["w"], b=s["b"])


# ---------------------------------------------------------------------- work

def work(case):
    """Each input read once and each output written once, and the method's own arithmetic."""
    c, kind = case, case["kind"]

    def ions(n, ndim, qs):  # the store read (28 / 32 bytes), the pushed store with its order written (28 / 32)
        return (56 if ndim == 2 else 64) * n, n * ((90 if not qs else 210) if ndim == 2 else (100 if not qs else 280))

    def fields(nc, nsub):  # E, B, n, J of two levels in, E, B, n, J out, cell_start
        return nc * (24 + 16 + 24 + 16 + 8), nc * (2 * nsub + 1) * 60

    if kind == "ensemble":
        b = f = 0
        for sp in _ens_specs(c, 0):
            nc = sp["side"] ** 2
            (b1, f1), (b2, f2) = ions(sp["ppc"] * nc, 2, True), fields(nc, 4)
            b, f = b + b1 + b2, f + f1 + f2
        return dict(bytes=b, flops=f)
    nz = c.get("nz", 1)
    nc, ndim = c["nx"] * c["ny"] * nz, 3 if nz > 1 else 2
    qs = c.get("shape", "qs") == "qs"
    if kind in ("step", "open"):
        (b1, f1), (b2, f2) = ions(c["ppc"] * nc, ndim, qs), fields(nc, c["nsub"])
        return dict(bytes=b1 + b2, flops=f1 + f2)
    if kind == "particles":
        b, f = ions(c["ppc"] * nc, ndim, qs)
        return dict(bytes=b + 4 * c["ppc"] * nc * 2 + 48 * nc, flops=f)
    if kind == "start":
        b, f = ions(c["ppc"] * nc, ndim, qs)
        return dict(bytes=b + 44 * nc, flops=f // 2)
    if kind == "fields":
        b, f = fields(nc, c["nsub"])
        return dict(bytes=b - 8 * nc - 16 * nc, flops=f)
    mac = 9 * (7 * 32 + 32 * 32 + 32 * 32 + 32 * 3)
    if kind == "predict":
        return dict(bytes=nc * (28 + 12), flops=2 * mac * nc)
    # forward, the weights' gradient of every layer and the data's of all but the first
    mac = 2 * mac + 9 * (32 * 32 + 32 * 32 + 32 * 3)
    return dict(bytes=nc * c["batch"] * 40 + 4 * 4 * 21600, flops=2 * mac * nc * c["batch"])


# --------------------------------------------------------------------- exact

class _Box:
    """The method in 64 bits on whole-grid tensors [nz, ny, nx]."""

    def __init__(self, cfg):
        self.c = cfg
        self.open = bool(cfg.open_x)
        self.shape = (cfg.nz, cfg.ny, cfg.nx)
        self.gamma, self.f32 = cfg.gamma_e, np.float32
        if self.open:
            i = torch.arange(cfg.nx, device=DEV)
            d = (torch.minimum(i, cfg.nx - 1 - i) - 1).clamp(min=0).double()
            w = max(cfg.buffer_cells, 1)
            self.eta_h = cfg.eta_h + cfg.eta_h_buffer * torch.where(d < cfg.buffer_cells, 1.0 - d / w, 0.0)
            self.inner = torch.ones(cfg.nx, device=DEV, dtype=torch.float64)
            self.inner[0] = self.inner[-1] = 0.0
        else:
            self.eta_h = cfg.eta_h

    def grid(self, F):
        return F.double().reshape(F.shape[:-1] + self.shape)

    def flat(self, F):
        return F.reshape(F.shape[:-3] + (-1,))

    def d(self, a, ax, ghost=False):
        h = (self.c.dx, self.c.dy, self.c.dz)[ax]
        r = (torch.roll(a, -1, -1 - ax) - torch.roll(a, 1, -1 - ax)) / (2 * h)
        return r * self.inner if ghost and self.open and ax == 0 else r

    def lap(self, a):
        r = 0.0
        for ax, h in enumerate((self.c.dx, self.c.dy, self.c.dz)):
            t = (torch.roll(a, -1, -1 - ax) + torch.roll(a, 1, -1 - ax) - 2 * a) / (h * h)
            r = r + (t * self.inner if self.open and ax == 0 else t)
        return r

    def curl(self, F, ghost=False):
        D = lambda a, ax: self.d(F[a], ax, ghost)  # noqa: E731
        return torch.stack([D(2, 1) - D(1, 2), D(0, 2) - D(2, 0), D(1, 0) - D(0, 1)])

    def fill(self, F):
        if self.open:
            F = F.clone()
            F[..., 0], F[..., -1] = F[..., 1], F[..., -2]
        return F

    def eos(self, n):
        c = self.c
        return c.n0 * c.te * (n.clamp(min=c.n_floor) / c.n0) ** c.gamma_e

    def ohm(self, B, n, J, p=None, B0=None):
        c = self.c
        nf = n.clamp(min=c.n_floor)
        p = self.eos(n) if p is None else p
        cur = self.curl(B, True)
        E = torch.linalg.cross((cur - J) / nf, B if B0 is None else B0 + B, dim=0)
        E = E - torch.stack([self.d(p, 0, True), self.d(p, 1), self.d(p, 2)]) / nf + c.eta * cur
        if self.open or c.eta_h:
            E = E - self.eta_h * torch.stack([self.lap(cur[a]) for a in range(3)])
        return E

    def rate(self, B, n, J, p):
        c, g = self.c, self.c.gamma_e
        nf = n.clamp(min=c.n_floor)
        u = (J - self.curl(B)) / nf
        div = sum(self.d(p * u[a], a) for a in range(3))
        adv = sum(u[a] * self.d(p, a) for a in range(3))
        return -g * div + (g - 1) * adv + (g - 1) * c.kappa0 * self.lap(p / nf)

    def advance(self, B, n, J, npv, Jp, p=None, B0=None):
        c = self.c
        h = c.dt / max(c.nsub, 1)
        faraday = lambda B, E, s: self.fill(B - s * self.curl(E))  # noqa: E731
        B = self.fill(B)
        for _ in range(c.nsub):
            Ea = self.ohm(B, n, J, p, B0)
            Bs = faraday(B, Ea, h / 2)
            ps = None if p is None else p + h / 2 * self.rate(B, n, J, p)
            Eb = self.ohm(Bs, n, J, ps, B0)
            if p is not None:
                p = p + h * self.rate(Bs, n, J, ps)
            B = faraday(B, Eb, h)
        n1, J1 = 1.5 * n - 0.5 * npv, 1.5 * J - 0.5 * Jp
        return B, self.ohm(B, n1, J1, p, B0), p

    def smooth(self, F):
        for _ in range(self.c.nsmooth):
            for ax in range(self.c.ndim):
                F = 0.25 * (torch.roll(F, 1, -1 - ax) + 2 * F + torch.roll(F, -1, -1 - ax))
        return F

    # ----- ions: index arrays and offsets in 64 bits, a slice of the store at a time

    def points(self, idx, off):
        """Cells and weights of the shape at the offsets."""
        c = self.c
        n = (c.nx, c.ny, c.nz)
        lin = lambda i: i[0] + c.nx * (i[1] + c.ny * i[2])  # noqa: E731
        if c.shape == W.SHAPE_NGP:
            return [(lin(idx), torch.ones_like(off[0]))]
        out, side = [], 0.0
        for a in range(c.ndim):
            for s in (1, -1):
                wt = (1 + s * off[a]) ** 2 / 12
                k = list(idx)
                k[a] = torch.remainder(idx[a] + s, n[a])
                out.append((lin(k), wt))
                side = side + wt
        return out + [(lin(idx), 1 - side)]

    def split(self, cell):
        c = self.c
        cell = cell.long()
        return [cell % c.nx, (cell // c.nx) % c.ny, cell // (c.nx * c.ny)]

    def shift(self, idx, off, vel, dt):
        c = self.c
        n, h = (c.nx, c.ny, c.nz), (c.dx, c.dy, c.dz)
        idx, off = list(idx), list(off)
        for a in range(c.ndim):
            x = off[a] + vel[a] * (2 * dt / h[a])
            s = torch.floor((x + 1) / 2)
            off[a] = x - 2 * s
            idx[a] = torch.remainder(idx[a] + s.long(), n[a])
        return idx, off

    def slices(self, p):
        n = p["cell"].numel()
        for a in range(0, n, 1 << 24):
            s = slice(a, min(n, a + (1 << 24)))
            yield s, self.split(p["cell"][s]), [p[k][s].double() for k in ("ox", "oy", "oz")[:self.c.ndim]], [p[k][s].double() for k in ("ux", "uy", "uz")]

    def deposit(self, acc, idx, off, vel, w):
        for cell, wt in self.points(idx, off):
            a = w * wt
            acc[0].index_add_(0, cell, a)
            for k in range(3):
                acc[1 + k].index_add_(0, cell, a * vel[k])

    def moments(self, acc):
        c = self.c
        m = self.fill((acc * (c.qs / (c.dx * c.dy * c.dz))).reshape((4,) + self.shape))
        return m[0], m[1:]

    def still(self, p):
        acc = torch.zeros((4, self.c.ncell), device=DEV, dtype=torch.float64)
        for s, idx, off, vel in self.slices(p):
            self.deposit(acc, idx, off, vel, p["w"][s].double())
        return self.moments(acc)

    def push(self, p, E, B):
        """(n, J at the mid-point, the new velocities in the store's order)."""
        c = self.c
        acc = torch.zeros((4, c.ncell), device=DEV, dtype=torch.float64)
        E, B = self.flat(E), self.flat(B)
        new = {k: torch.empty(p["cell"].numel(), device=DEV, dtype=torch.float64) for k in ("ux", "uy", "uz")}
        a = 0.5 * c.qs / c.ms * c.dt
        for s, idx, off, vel in self.slices(p):
            e, b = 0.0, 0.0
            for cell, wt in self.points(idx, off):
                e, b = e + wt * E[:, cell], b + wt * B[:, cell]
            v = torch.stack(vel) + a * e
            t = a * b
            q = v + torch.linalg.cross(v, t, dim=0)
            v = v + torch.linalg.cross(q, 2 * t / (1 + (t * t).sum(0)), dim=0) + a * e
            for k, name in enumerate(new):
                new[name][s] = v[k]
            idx, off = self.shift(idx, off, v, 0.5 * c.dt)
            self.deposit(acc, idx, off, v, p["w"][s].double())
        return (*self.moments(acc), new)


def _blank(p, **kw):
    """The store's outputs: a value for those given, none for the rest."""
    return {k: kw.get(k) for k in p}


def _exact_step(cfg, p, B, gather_map):
    """One step of GpuSim from its initial state."""
    x = _Box(cfg)
    order = torch.argsort(p["cell"], stable=True)
    p = {k: v[order] for k, v in p.items()}
    B = x.grid(B)
    n0, J0 = x.still(p)
    n0, J0 = x.smooth(n0), x.smooth(J0)
    pe = x.eos(n0) if cfg.energy_eq else None
    E = x.ohm(B, n0, J0, pe)
    n, J, new = x.push(p, x.smooth(E), x.smooth(B))
    n, J = x.smooth(n), x.smooth(J)
    B, E, pe = x.advance(B, n, J, n0, J0, pe)
    out = dict(E=x.flat(E), B=x.flat(B), n=x.flat(n), J=x.flat(J), cell_start=None)
    # the moved store's order hangs on the cells; the mapped one keeps the order before the step
    out["store"] = _blank(p, **new, w=p["w"].double()) if gather_map else _blank(p)
    if gather_map:
        out["map"] = None
    if pe is not None:
        out["pe"] = x.flat(pe)
    return out


def _conv(X, w, ny, nx):
    """Periodic 3x3 layer on X [S, ny, nx, Cin], w [Cout, 9, Cin]."""
    cols = torch.cat([torch.roll(X, (1 - t // 3, 1 - t % 3), (1, 2)) for t in range(9)], dim=-1)
    return cols.reshape(-1, cols.shape[-1]) @ w.reshape(w.shape[0], -1).T


def _forward(params, norm, B, n, J, ny, nx):
    X = torch.stack([B[:, 0], B[:, 1], B[:, 2], n, J[:, 0], J[:, 1], J[:, 2]], dim=-1)
    X = ((X - norm[0]) / norm[1]).reshape(-1, ny, nx, 7)
    for k, (w, b) in enumerate(params):
        X = _conv(X, w, ny, nx) + b
        X = (torch.tanh(X) if k < 3 else X).reshape(-1, ny, nx, w.shape[0])
    return X.reshape(X.shape[0], ny * nx, 3).transpose(1, 2)


def _exact_net(c, seed, g):
    cfg, wts, norm, data, idx = _net(c, seed, g)
    f64 = lambda a: torch.tensor(np.asarray(a, np.float32), device=DEV, dtype=torch.float64)  # noqa: E731
    params = [(f64(w), f64(b)) for w, b in wts]
    norm = tuple(f64(a) for a in norm)
    B, n, J, Bt = (t.double() for t in data)
    if c["kind"] == "predict":
        return (B + norm[2][:, None] * _forward(params, norm, B, n, J, cfg.ny, cfg.nx))[0]
    flat = [t.requires_grad_() for w, b in params for t in (w, b)]
    m, v = [torch.zeros_like(t) for t in flat], [torch.zeros_like(t) for t in flat]
    for k in range(TRAIN_WARM + 1):
        gsum = [torch.zeros_like(t) for t in flat]
        for s in idx[k].tolist():
            d = _forward(params, norm, B[s:s + 1], n[s:s + 1], J[s:s + 1], cfg.ny, cfg.nx)
            loss = ((d - (Bt[s:s + 1] - B[s:s + 1]) / norm[2][:, None]) ** 2).sum() / (3.0 * cfg.ncell * idx.shape[1])
            for a, q in zip(gsum, torch.autograd.grad(loss, flat)):
                a += q
        for a in range(len(flat)):
            m[a] = 0.9 * m[a] + 0.1 * gsum[a]
            v[a] = 0.999 * v[a] + 0.001 * gsum[a] ** 2
    c1, c2 = 1 - 0.9 ** (TRAIN_WARM + 1), 1 - 0.999 ** (TRAIN_WARM + 1)
    new = [(t - TRAIN_LR * (a / c1) / ((b / c2).sqrt() + 1e-8)).detach() for t, a, b in zip(flat, m, v)]
    return dict(w=torch.cat([t.reshape(-1) for t in new[0::2]]), b=torch.cat([t.reshape(-1) for t in new[1::2]]))


def exact(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind == "ensemble":
        out = []
        for cfg, p, B in [_ens_run(sp, g) for sp in _ens_specs(c, seed)]:
            r = _exact_step(cfg, p, B, True)
            out.append({k: r[k] for k in ("E", "B", "n", "J")})
        return out
    if kind in ("predict", "train"):
        return _exact_net(c, seed, g)
    cfg = _config(c)
    x = _Box(cfg)
    if kind == "step":
        return _exact_step(cfg, _ions(cfg, c["flavour"], c["ppc"], g), _field(cfg, c["flavour"]), c["gather_map"])
    if kind == "open":
        p, B1 = _ions(cfg, "wind", c["ppc"] * (cfg.nx - 2) / cfg.nx, g), x.fill(x.grid(_field(cfg, "wind")))
        p["w"].fill_(cfg.dx * cfg.dy * cfg.dz / c["ppc"])
        B0 = torch.zeros_like(B1)
        B0[1] = 1.0
        n0, J0 = x.still(p)
        E = x.ohm(B1, n0, J0, None, B0)
        n, J, _ = x.push(p, E, B0 + B1)
        B1, E, _ = x.advance(B1, n, J, n0, J0, None, B0)
        return dict(E=x.flat(E), B1=x.flat(B1), B=x.flat(B0 + B1), n=x.flat(n), J=x.flat(J), cell_start=None)
    if kind == "particles":
        p, perm, _ = _moved(cfg, c, g)
        p = {k: v[perm.long()] for k, v in p.items()}
        E, B = _eb(cfg, g)
        n, J, new = x.push(p, x.grid(E), x.grid(B))
        return dict(store=_blank(p, **new, w=p["w"]), n=x.flat(n), J=x.flat(J), map=None, cell_start=None)
    if kind == "start":
        p = _ions(cfg, "harris", c["ppc"], g)
        order = torch.argsort(p["cell"], stable=True)
        p = {k: v[order] for k, v in p.items()}
        n, J = x.still(p)
        E = x.ohm(x.grid(_field(cfg, "harris")), n, J)
        return dict(store=dict(_blank(p, **p), cell=None), cell_start=None, n=x.flat(n), J=x.flat(J), E=x.flat(E))
    _, B = _eb(cfg, g)
    n, J, npv, Jp = (x.grid(t) for t in _moments(cfg, g))
    B, E, _ = x.advance(x.grid(B), n, J, npv, Jp)
    return dict(B=x.flat(B), E=x.flat(E))


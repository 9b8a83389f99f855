"""Timed workloads of the library, over the range that programs use it in.

Five kinds of case, each one pass through the public entry points:

* ``step``     : one SSP-RK3 step (three fused stages) by ``solver.Stepper``,
                 replayed from its HIP graph.  The step always starts from the
                 initial state, so every pass does the same work.
* ``rhs``      : the right-hand side by the separate calls (scatter, element
                 right-hand side, assembly, gather, finalize) and the stage
                 combination, as a program with its own time integrator calls
                 them.
* ``boundary`` : what an adaptive run evaluates between two steps: criterion
                 flags, maximum wind, forecaster features, network, merged
                 flags.
* ``transfer`` : the solution moved onto an adapted layout.
* ``train``    : one mini-batch of the forecaster's training (gradient, Adam).

The meshes are those of the benchmark and of the tests (64 x 64 x 16 on
1000 km, 64 x 64 x 8 base on 400 km with one or two refined levels, 8 x 8 x 4)
and ragged ones; the states are balanced vortices with smooth perturbations.
``exact`` evaluates the same discretisation with plain torch in FP64.
"""

import math

import numpy as np
import torch
from numpy.polynomial import legendre

from paper_2410_21607_amd import api
from paper_2410_21607_amd.solver import Stepper

PHYS = dict(f=5e-5, g=9.81, R_d=287.0, c_p=1004.0, p00=1.0e5)
RK3 = ((0.0, 1.0, 1.0), (0.75, 0.25, 0.25), (1.0 / 3.0, 2.0 / 3.0, 2.0 / 3.0))
THRESHOLDS = (2e-4, 1e-3)          # vertical vorticity [1/s], levels 1 and 2
SCALE = np.array([1.0, 1e3, 1e3, 0.05, 1.0, 1.0, 1.0, 20.0, 1e3, 1e4, 1e3, 1e3, 0.05, 0.5, 1e4,
                  1.0], dtype=np.float32)
ROWS = 200000                      # training samples, as the forecaster experiment draws
DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _mesh(N, nx, ny, nz, L=400e3, H=20e3, levels=0, radius=0.135, periodic=True, precision="fp64",
          terrain=0.0, cs=0.0, tuned=False):
    """Plain description of a mesh and of the options of its stage: ``radius``
    (of the shorter side) is the disc refined once, columns well inside it are
    refined again when levels = 2; ``tuned`` lets the autotuner pick the
    layout, as the benchmark does (an adaptive run takes the default)."""
    return dict(N=N, nx=nx, ny=ny, nz=nz, L=L, H=H, levels=levels, radius=radius,
                periodic=periodic, precision=precision, terrain=terrain, cs=cs, tuned=tuned)


def listed():
    bench = dict(N=4, nx=64, ny=64, nz=16, L=1000e3, H=25e3, tuned=True)
    amr2 = dict(nx=64, ny=64, nz=8, levels=1)
    return [
        # the smallest workload (256 elements): launches and latency decide
        dict(name="step_8x8x4_n4", kind="step", **_mesh(4, 8, 8, 4)),
        # the throughput workload of the benchmark, and its FP32 variant
        dict(name="step_64x64x16_n4", kind="step", **_mesh(**bench)),
        dict(name="step_64x64x16_n4_fp32", kind="step", **_mesh(**bench, precision="fp32")),
        # the same with the sub-grid and absorbing-layer terms of long runs
        dict(name="step_64x64x16_n4_dissipation", kind="step", **_mesh(**bench, cs=0.21)),
        # two-level AMR: the layout an adaptive run steps on (default tuning),
        # the high order, and terrain-following coordinates
        dict(name="step_amr2_n4", kind="step", **_mesh(4, **amr2)),
        dict(name="step_amr2_n7", kind="step", **_mesh(7, **amr2, tuned=True)),
        dict(name="step_amr2_n4_terrain", kind="step", **_mesh(4, **amr2, terrain=2000.0, tuned=True)),
        # ragged counts, walls instead of periodic sides, another order
        dict(name="step_37x29x5_n5_walls", kind="step", **_mesh(5, 37, 29, 5, periodic=False)),
        # the separate calls on the two-level mesh
        dict(name="rhs_amr2_n4", kind="rhs", **_mesh(4, **amr2)),
        # one adaptation boundary of the three-level run with the forecaster,
        # and the transfer of its state to the next layout
        dict(name="boundary_amr3_n4", kind="boundary", **_mesh(4, 64, 64, 8, levels=2, radius=0.125)),
        dict(name="transfer_amr3_n4", kind="transfer", shift=0.02,
             **_mesh(4, 64, 64, 8, levels=2, radius=0.125)),
        # one training step at the forecaster's batch size
        dict(name="train_batch1024", kind="train", batch=1024),
    ]


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["rhs", "boundary", "transfer", "train", "train"])
    if kind == "train":
        return dict(kind=kind, batch=int(round(math.exp(rng.uniform(math.log(33), math.log(4097))))))
    N = rng.choice([1, 2, 3, 3, 4, 4, 4, 5, 5, 6, 7, 8])
    nz = rng.randint(2, 20)
    levels = rng.choice([0, 0, 1, 2])
    # unique nodes from 2e4 to 3e6, log-uniform; a few more on refined meshes
    nodes = math.exp(rng.uniform(math.log(2e4), math.log(3e6)))
    side = max(6.0, math.sqrt(nodes / (N * N * (nz * N + 1) * (1 + 0.3 * levels))))
    nx = max(6, min(160, int(side * rng.uniform(0.8, 1.25))))
    ny = max(6, min(160, int(side * side / nx)))
    m = dict(levels=levels, radius=rng.uniform(0.11, 0.16), periodic=rng.random() < 0.7)
    if kind == "step":
        m.update(precision=rng.choice(["fp64", "fp64", "fp32"]), tuned=rng.random() < 0.5)
        extra = rng.random()
        if extra < 0.2:
            m.update(terrain=rng.uniform(300.0, 2500.0))
        elif extra < 0.35:
            m.update(cs=0.21)
    elif kind == "rhs":
        m.update(precision=rng.choice(["fp64", "fp32"]))
    case = dict(kind=kind, **_mesh(N, nx, ny, nz, **m))
    if kind == "transfer":
        # the vortex moves by up to a column and a half between two layouts
        case.update(levels=max(1, levels), shift=rng.uniform(0.4, 1.5) / nx)
    return case


# ------------------------------------------------------------------ inputs
def _columns(case, shift=0.0):
    """(n, 3) columns (level, ix, iy) in Morton order: the base grid, refined
    inside a disc about the vortex (moved by ``shift`` sides along x)."""
    nx, ny, L = case["nx"], case["ny"], case["L"]
    Ly = L * ny / nx
    d0 = max(L / nx, Ly / ny)
    radii = [case["radius"] * min(L, Ly)]
    radii.append(radii[0] - 2.0 * d0)
    ix, iy = (a.ravel() for a in np.meshgrid(np.arange(nx), np.arange(ny), indexing="ij"))
    leaves, level = [], 0
    while True:
        dx, dy = L / (nx << level), Ly / (ny << level)
        # nearest point of the column to the disc's centre
        px = np.maximum(np.abs(-0.5 * L + (ix + 0.5) * dx - shift * L) - 0.5 * dx, 0.0)
        py = np.maximum(np.abs(-0.5 * Ly + (iy + 0.5) * dy) - 0.5 * dy, 0.0)
        split = np.zeros(ix.size, bool)
        if level < case["levels"] and radii[level] > 0:
            split = np.hypot(px, py) < radii[level]
        leaves.append(np.stack([np.full((~split).sum(), level), ix[~split], iy[~split]], axis=1))
        if not split.any():
            break
        sx, sy = ix[split], iy[split]
        ix = np.concatenate([2 * sx, 2 * sx + 1, 2 * sx, 2 * sx + 1])
        iy = np.concatenate([2 * sy, 2 * sy, 2 * sy + 1, 2 * sy + 1])
        level += 1
    cols = np.concatenate(leaves)
    key = np.zeros(len(cols), np.int64)
    fx, fy = cols[:, 1] << (level - cols[:, 0]), cols[:, 2] << (level - cols[:, 0])
    for b in range(20):
        key |= ((fx >> b) & 1) << (2 * b) | ((fy >> b) & 1) << (2 * b + 1)
    return cols[np.argsort(key, kind="stable")]


def _mesh_case(case, shift=0.0):
    return dict(N=case["N"], nx0=case["nx"], ny0=case["ny"], columns=_columns(case, shift),
                Lx=case["L"], Ly=case["L"] * case["ny"] / case["nx"],
                z_edges=np.linspace(0.0, case["H"], case["nz"] + 1),
                periodic_x=case["periodic"], periodic_y=case["periodic"], phys=PHYS)


def _reference(z):
    """Hydrostatic atmosphere of constant N_bv = 0.01 1/s over 300 K."""
    p = PHYS
    n2, ts, cv = 1e-4, 300.0, p["c_p"] - p["R_d"]
    th = ts * torch.exp(n2 * z / p["g"])
    pi = 1.0 + p["g"] ** 2 / (p["c_p"] * ts * n2) * (torch.exp(-n2 * z / p["g"]) - 1.0)
    rho = p["p00"] * pi ** (cv / p["R_d"]) / (p["R_d"] * th)
    dth = th * n2 / p["g"]
    drho = rho * ((cv / p["R_d"]) * (-p["g"] / (p["c_p"] * th)) / pi - dth / th)
    return dict(rho0=rho, theta0=th, dth=dth, drho=drho, p0=p["p00"] * pi ** (p["c_p"] / p["R_d"]))


def _modes(rng, x, y, z, Lx, Ly, H):
    out = torch.zeros_like(x)
    for _ in range(5):
        k = rng.integers(1, 5, size=2)
        ph = rng.uniform(0, 2 * np.pi, size=2)
        out += rng.uniform(0.1, 0.3) * torch.cos(2 * np.pi * k[0] * x / Lx + ph[0]) \
            * torch.cos(2 * np.pi * k[1] * y / Ly + ph[1]) \
            * torch.sin(float(rng.integers(1, 3)) * np.pi * z / H)
    return out


def _state(case, seed, x, y, z, moved=0.0):
    """(5, ...) perturbation state of a balanced vortex of 25 to 40 m/s at the
    points (x, y, z): gradient-wind p', hydrostatic rho', theta' from the
    equation of state, smooth seeded perturbations of theta' (0.3 K at fixed
    pressure) and w, a uniform steering wind.  ``moved`` [m]: along x."""
    p, rng = PHYS, np.random.default_rng(seed)
    L, Ly, H = case["L"], case["L"] * case["ny"] / case["nx"], case["H"]
    S = min(L, Ly)
    vmax, rmax = rng.uniform(25.0, 40.0), rng.uniform(0.05, 0.08) * S
    cx, cy = rng.uniform(-0.02, 0.02, size=2) * S
    rt = torch.linspace(0.0, 0.5 * S, 20001, dtype=torch.float64, device=x.device)
    wind = lambda r: 2.0 * vmax * (r / rmax) / (1.0 + (r / rmax) ** 2) * torch.exp(-(4.0 * r / S) ** 6)
    vt = wind(rt)
    fa = torch.where(rt > 0, vt * vt / rt.clamp(min=1e-30), torch.zeros_like(rt)) + 0.0
    def inward(f):
        c = torch.cumsum(0.5 * (rt[1:] - rt[:-1]) * (f[1:] + f[:-1]), 0)
        return torch.cat([c[-1:], c[-1] - c])
    def interp(tab, r):
        s = (r / (rt[1] - rt[0])).clamp(max=rt.numel() - 1.0)
        i = s.floor().long().clamp(max=rt.numel() - 2)
        return tab[i] + (s - i) * (tab[i + 1] - tab[i])
    xr, yr = x - cx - moved, y - cy
    r = torch.hypot(xr, yr)
    A, B = interp(inward(fa), r), interp(inward(vt), r)
    zv = (1.0 - z / (0.75 * H)).clamp(min=0.0)
    dzv = torch.where(z < 0.75 * H, -1.0 / (0.75 * H), 0.0).to(x)
    bg = _reference(z)
    Sr, dS = zv * zv * A + p["f"] * zv * B, 2.0 * zv * dzv * A + p["f"] * dzv * B
    pres = bg["p0"] - bg["rho0"] * Sr
    rho = bg["rho0"] + (bg["drho"] * Sr + bg["rho0"] * dS) / p["g"]
    th = p["p00"] / (p["R_d"] * rho) * (pres / p["p00"]) ** ((p["c_p"] - p["R_d"]) / p["c_p"])
    dth = 0.3 * _modes(rng, x, y, z, L, Ly, H)
    spin = wind(r) * zv / r.clamp(min=1e-30)
    return torch.stack([rho * th / (th + dth) - bg["rho0"], 5.0 - spin * yr, spin * xr,
                        0.2 * _modes(rng, x, y, z, L, Ly, H), th + dth - bg["theta0"]])


def _surface(case, x, y):
    """Terrain height: a Gaussian mountain of a tenth of the shorter side."""
    w = 0.1 * min(case["L"], case["L"] * case["ny"] / case["nx"])
    return case["terrain"] * torch.exp(-(x * x + y * y) / (w * w))


def _time_step(case):
    N, deep = case["N"], max(case["levels"], 0)
    x = _lgl(N)[0]
    gap = 0.5 * (x[1] - x[0])
    h = min(gap * case["H"] / case["nz"] * (1.0 - case["terrain"] / case["H"]),
            gap * case["L"] / (case["nx"] << deep))
    return 0.4 * h / 390.0


def _points(case, hxy, z):
    """x, y, z of the nodes [h][kz] (physical heights) and the surface."""
    hx, hy = hxy[:, 0], hxy[:, 1]
    zs = _surface(case, hx, hy) if case["terrain"] else torch.zeros_like(hx)
    zp = z[None, :] + zs[:, None] * (1.0 - z[None, :] / case["H"])
    return hx[:, None].expand_as(zp), hy[:, None].expand_as(zp), zp, zs


def _setup(case, seed, shift=0.0, moved=0.0, n_states=1):
    """Mesh with its reference state, terrain and dissipation, and padded
    states on it (the later ones with the vortex moved on)."""
    mesh = api.Mesh.from_case(_mesh_case(case, shift))
    hxy, _, z = mesh.coords()
    hxy, zt = (torch.as_tensor(a, device=DEV) for a in (hxy, z))
    flat = _reference(torch.as_tensor(z))
    mesh.set_reference(*(flat[k].numpy() for k in ("rho0", "theta0", "dth")))
    x, y, zp, zs = _points(case, hxy, zt)
    if case["terrain"]:
        ref = _reference(zp)
        mesh.set_terrain(zs.cpu().numpy(), *(ref[k].cpu().numpy() for k in ("rho0", "theta0", "dth")))
    if case["cs"]:
        mesh.set_dissipation(case["cs"], 1.0, 4000.0)
    states = []
    for k in range(n_states):
        q = mesh.state().view(5, mesh.info["n_h"], mesh.ldz)
        q[:, :, :z.size] = _state(case, seed, x, y, zp, moved - 1500.0 * k)
        states.append(q.reshape(-1))
    return mesh, states


def _network(seed):
    g = torch.Generator().manual_seed(seed)
    parts = []
    for n_out, n_in in ((64, 16), (64, 64), (3, 64)):
        parts += [torch.randn(n_out * n_in, generator=g) / math.sqrt(n_in), 0.1 * torch.randn(n_out, generator=g)]
    return torch.cat(parts)


def _samples(seed, batch):
    g = torch.Generator().manual_seed(seed)
    X = torch.randn(ROWS, 16, generator=g)
    Y = torch.randint(0, 3, (ROWS,), generator=g, dtype=torch.int8)
    idx = torch.randint(0, ROWS, (8, batch), generator=g, dtype=torch.int32)
    return X, Y, idx


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        X, Y, idx = _samples(seed, case["batch"])
        net = _network(seed).cuda()
        return dict(kind=kind, X=X.cuda(), Y=Y.cuda(), idx=list(idx.cuda()), t=0, net=net,
                    m=torch.zeros_like(net), v=torch.zeros_like(net), grad=torch.zeros_like(net),
                    loss=torch.zeros(1, device="cuda"),
                    work=torch.empty(case["batch"] * api.MLP_WORK, device="cuda"))
    prec = api.SEM_FP32 if case["precision"] == "fp32" else api.SEM_FP64
    if kind == "step":
        mesh, (q,) = _setup(case, seed)
        if case["tuned"]:
            api.sem_stage_autotune(mesh, q, q.clone(), torch.zeros_like(q), prec, reps=5)
        return dict(kind=kind, stepper=Stepper(mesh, q, _time_step(case), prec, graph=True))
    if kind == "rhs":
        mesh, (q,) = _setup(case, seed)
        new = lambda n: torch.zeros(max(n, 1), dtype=torch.float64, device="cuda")
        return dict(kind=kind, mesh=mesh, q=q, prec=prec, dt=_time_step(case), hv=new(mesh.n_hstate),
                    rE=new(5 * mesh.n_local), acc=mesh.state(), c=new(mesh.n_hstate), r=mesh.state(),
                    out=mesh.state())
    if kind == "transfer":
        mesh, (q,) = _setup(case, seed)
        new = api.Mesh.from_case(_mesh_case(case, case["shift"]))
        return dict(kind=kind, transfer=api.Transfer(mesh, new), q=q, out=new.state())
    mesh, (q, q_prev) = _setup(case, seed, n_states=2)
    ne, nc, lvl = mesh.info["n_elem"], mesh.info["n_col"], max(case["levels"], 1)
    i8 = lambda n: torch.empty(n, dtype=torch.int8, device="cuda")
    L, Ly = case["L"], case["L"] * case["ny"] / case["nx"]
    return dict(kind=kind, mesh=mesh, q=q, q_prev=q_prev, lvl=lvl, thr=np.array(THRESHOLDS[:lvl]),
                plain=i8(ne), plain_col=i8(nc), dem=i8(ne), flags=i8(ne), flags_col=i8(nc),
                feat=torch.empty(ne * 16, device="cuda"), logits=torch.empty(ne * 3, device="cuda"),
                wind=torch.zeros(1, dtype=torch.float64, device="cuda"), net=_network(seed).cuda(),
                box=(-0.5 * L, 0.5 * L, -0.5 * Ly, 0.5 * Ly))


def run(state):
    s = state
    kind = s["kind"]
    if kind == "step":
        s["stepper"].cur = 0          # the step always starts from the first buffer
        return s["stepper"].step(1)
    if kind == "rhs":
        m = s["mesh"]
        if m.n_hang:
            api.sem_nc_project(m, api.SEM_SCATTER, s["q"], s["hv"])
        api.sem_rhs(m, s["q"], s["hv"] if m.n_hang else None, s["rE"], s["prec"])
        api.sem_dss(m, api.SEM_ASSEMBLE, rE=s["rE"], acc=s["acc"], c=s["c"] if m.n_hang else None)
        if m.n_hang:
            api.sem_nc_project(m, api.SEM_GATHER, s["c"], s["acc"])
        api.sem_dss(m, api.SEM_FINALIZE, acc=s["acc"], r=s["r"])
        api.sem_stage_update(m, 0.75, 0.25, 0.25 * s["dt"], s["q"], s["q"], s["r"], s["out"])
        return [s["r"], s["out"]]
    if kind == "transfer":
        api.sem_transfer_apply(s["transfer"], s["q"], s["out"])
        return s["out"]
    if kind == "boundary":
        m, crit = s["mesh"], api.SEM_CRIT_VORTZ
        api.amr_flag(m, s["q"], crit, s["thr"], s["lvl"], s["plain"], s["plain_col"])
        api.sem_max_wind(m, s["q"], s["box"], s["wind"])
        api.amr_features(m, s["q"], s["q_prev"], s["plain"], crit, s["thr"], s["lvl"], SCALE,
                         s["feat"], s["dem"])
        api.mlp_forward(s["net"], s["feat"].view(-1, 16), s["logits"])
        api.amr_forecast_flags(m, s["logits"], s["plain"], s["lvl"], s["flags"], s["flags_col"])
        return {k: s[k] for k in ("plain", "plain_col", "wind", "feat", "dem", "logits", "flags",
                                  "flags_col")}
    s["t"] += 1
    api.mlp_backward(s["net"], s["X"], s["Y"], s["idx"][(s["t"] - 1) % len(s["idx"])], s["work"],
                     s["grad"], s["loss"])
    api.mlp_adam_step(s["net"], s["grad"], s["m"], s["v"], s["t"])
    return [s["grad"], s["loss"], s["net"], s["m"], s["v"]]


def work(case):
    """Bytes and floating-point operations that one pass cannot do without."""
    kind = case["kind"]
    if kind == "train":
        n, P = case["batch"], api.MLP_NPARAM
        # parameters and moments read and written, gradient written, samples read
        return dict(bytes=4 * P * 7 + n * (64 + 1 + 4), flops=6.0 * n * 5312)
    info = api.sem_mesh_plan(_mesh_case(case))[0]
    nodes, local, hang = info["n_dof"], info["n_local"], info["n_hang"]
    # per local node: 18 derivatives of N + 1 taps, pressure and the terms
    rhs = local * (36.0 * (case["N"] + 1) + 90.0)
    if kind == "step":
        # q_s, q^n (stages 2 and 3) and q_out, 5 fields; with terrain the
        # reference of every node
        per = 2 * 3 + 2 + (3 * 5 / 5.0 if case["terrain"] else 0.0)
        extra = local * 3 * (30.0 * (case["N"] + 1) + 40.0) if case["cs"] else 0.0
        return dict(bytes=40.0 * nodes * per, flops=3.0 * rhs + extra)
    if kind == "rhs":
        # each call's own arrays: q, hanging values; q -> rE; rE -> acc, c;
        # c -> acc; acc -> r; q^n, q_s, r -> q_out
        return dict(bytes=40.0 * (8 * nodes + 2 * local + 5 * hang), flops=rhs)
    if kind == "transfer":
        new = api.sem_mesh_plan(_mesh_case(case, case["shift"]))[0]["n_dof"]
        return dict(bytes=40.0 * (nodes + new), flops=10.0 * new)
    ne = info["n_elem"]
    # flags: u, v; wind: u, v; features: five fields and the earlier u, v;
    # features written and read, logits, flags
    return dict(bytes=8.0 * nodes * 11 + ne * (64 * 2 + 12 * 2 + 6),
                flops=local * (36.0 * case["N"] + 200.0) + ne * 2.0 * 5312)


# ------------------------------------------------- the same in plain FP64
def _lgl(N):
    """LGL nodes, weights and derivative matrix (numpy)."""
    c = np.zeros(N + 1)
    c[N] = 1.0
    d1, d2 = legendre.legder(c), legendre.legder(c, 2)
    xi = legendre.legroots(d1) if N > 1 else np.zeros(0)
    for _ in range(3):
        if N > 1:
            xi = xi - legendre.legval(xi, d1) / legendre.legval(xi, d2)
    x = np.concatenate([[-1.0], np.sort(xi), [1.0]])
    P = legendre.legval(x, c)
    D = np.zeros((N + 1, N + 1))
    for i in range(N + 1):
        for j in range(N + 1):
            if i != j:
                D[i, j] = P[i] / P[j] / (x[i] - x[j])
    D[np.arange(N + 1), np.arange(N + 1)] = -D.sum(axis=1)
    return x, 2.0 / (N * (N + 1) * P * P), D


def _lagrange(x, s):
    """l_m(s) of the nodes x, (len(s), len(x))."""
    out = torch.ones(s.numel(), x.numel(), dtype=torch.float64, device=s.device)
    for m in range(x.numel()):
        for k in range(x.numel()):
            if k != m:
                out[:, m] *= (s - x[k]) / (x[m] - x[k])
    return out


class _Plain:
    """A column mesh in plain torch: values of unique nodes to element-local
    ones (hanging points take the coarse face's polynomial) and back."""

    def __init__(self, case, shift=0.0):
        self.case, mc = case, _mesh_case(case, shift)
        # only the numbering of the unique nodes is the library's
        info, hxy, _, z, _ = api.sem_mesh_plan(mc)
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=DEV)
        N, self.Lx, self.Ly = case["N"], mc["Lx"], mc["Ly"]
        self.N, self.np1, self.nz, self.nzn, self.ldz = N, N + 1, case["nz"], info["nzn"], info["ldz"]
        x, w, D = _lgl(N)
        self.x, self.w, self.D = t(x), t(w), t(D)
        self.hxy, self.z, self.n_h = t(hxy), t(z), info["n_h"]
        cols = t(mc["columns"])
        self.lev, self.ix, self.iy = cols[:, 0], cols[:, 1], cols[:, 2]
        self.nc = cols.shape[0]
        side = 2.0 ** self.lev.double()
        self.dx, self.dy = self.Lx / case["nx"] / side, self.Ly / case["ny"] / side
        self.x0, self.y0 = -0.5 * self.Lx + self.ix * self.dx, -0.5 * self.Ly + self.iy * self.dy
        s = 0.5 * (self.x + 1.0)
        px = (self.x0[:, None, None] + s[None, None, :] * self.dx[:, None, None]).expand(-1, N + 1, -1)
        py = (self.y0[:, None, None] + s[None, :, None] * self.dy[:, None, None]).expand(-1, -1, N + 1)
        px, py = px.reshape(self.nc, -1), py.reshape(self.nc, -1)
        key, keys = self._key(px, py), self._key(self.hxy[:, 0], self.hxy[:, 1])
        keys, order = torch.sort(keys)
        at = torch.searchsorted(keys, key).clamp(max=keys.numel() - 1)
        self.h = torch.where(keys[at] == key, order[at], -1)     # (nc, np1^2)
        self.hang = []                                           # per level: slots, coarse column, weights
        top = int(self.lev.max())
        for l in range(1, top + 1):
            c, p = torch.nonzero((self.h < 0) & (self.lev[:, None] == l), as_tuple=True)
            if c.numel() == 0:
                continue
            nx, ny = case["nx"] << (l - 1), case["ny"] << (l - 1)
            grid = torch.full((nx, ny), -1, dtype=torch.long, device=DEV)
            sel = torch.nonzero(self.lev == l - 1)[:, 0]
            grid[self.ix[sel], self.iy[sel]] = sel
            cw, ch = self.Lx / nx, self.Ly / ny
            coarse = torch.full_like(c, -1)
            for ox in (-0.01, 0.01):
                for oy in (-0.01, 0.01):
                    gx = torch.floor((px[c, p] + 0.5 * self.Lx) / cw + ox).long()
                    gy = torch.floor((py[c, p] + 0.5 * self.Ly) / ch + oy).long()
                    ok = (gx >= 0) & (gx < nx) & (gy >= 0) & (gy < ny) | case["periodic"]
                    coarse = torch.where((coarse < 0) & ok, grid[gx % nx, gy % ny], coarse)
            off = lambda a, a0, d, P: torch.remainder(a - a0 + 0.25 * d, P) - 0.25 * d
            sx = 2.0 * off(px[c, p], self.x0[coarse], cw, self.Lx) / cw - 1.0
            sy = 2.0 * off(py[c, p], self.y0[coarse], ch, self.Ly) / ch - 1.0
            wgt = _lagrange(self.x, sy)[:, :, None] * _lagrange(self.x, sx)[:, None, :]
            self.hang.append((c, p, coarse, wgt.reshape(c.numel(), -1)))
        self.kidx = torch.arange(self.nz, device=DEV)[:, None] * N + torch.arange(N + 1, device=DEV)[None, :]
        self.dz = t(np.diff(mc["z_edges"]))
        self.zs = None

    def _key(self, x, y):
        def one(a, L):
            if self.case["periodic"]:
                a = torch.remainder(a + 0.5 * L, L)
                a = torch.where(a >= L - 1e-6, a - L, a) - 0.5 * L
            return torch.round(a * 1e3).long()
        return one(x, self.Lx) * (1 << 32) + one(y, self.Ly)

    def scatter(self, q):
        """(F, n_h, K) -> (F, nc, np1^2, K)"""
        out = q[:, self.h.clamp(min=0)]
        for c, p, coarse, wgt in self.hang:
            out[:, c, p] = (wgt[None, :, :, None] * out[:, coarse]).sum(2)
        return out

    def gather(self, con):
        """The transpose of scatter."""
        con = con.clone()
        F, K = con.shape[0], con.shape[-1]
        for c, p, coarse, wgt in reversed(self.hang):
            v = con[:, c, p]
            con[:, c, p] = 0.0
            con.index_add_(1, coarse, wgt[None, :, :, None] * v[:, :, None, :])
        ok = self.h.reshape(-1) >= 0
        out = torch.zeros(F, self.n_h, K, dtype=torch.float64, device=DEV)
        return out.index_add_(1, self.h.reshape(-1)[ok], con.reshape(F, -1, K)[:, ok])

    def elements(self, loc):
        """(F, nc, np1^2, nzn) -> (F, nc, j, i, layer, k)"""
        e = loc[..., self.kidx]
        return e.reshape(loc.shape[0], self.nc, self.np1, self.np1, self.nz, self.np1)

    def from_elements(self, e):
        out = torch.zeros(e.shape[0], self.nc, self.np1 ** 2, self.nzn, dtype=torch.float64, device=DEV)
        e = e.reshape(e.shape[0], self.nc, self.np1 ** 2, self.nz, self.np1)
        for l in range(self.nz):
            out[..., l * self.N:l * self.N + self.np1] += e[..., l, :]
        return out

    def along(self, f, dim):
        return torch.tensordot(f, self.D, dims=([dim], [1])).movedim(-1, dim)

    def col(self, a):
        return a[:, None, None, None, None]

    def grad(self, f):
        """Physical derivatives of one field (nc, j, i, layer, k)."""
        fx = self.along(f, 2) * self.col(2.0 / self.dx)
        fy = self.along(f, 1) * self.col(2.0 / self.dy)
        fz = self.along(f, 4) * (2.0 / self.dz)[:, None]
        if self.zs is not None:
            fx, fy, fz = fx + self.ax * fz, fy + self.ay * fz, self.gs * fz
        return fx, fy, fz

    def setup(self):
        """Reference state, terrain metrics and masses."""
        case = self.case
        x, y, zp, zs = _points(case, self.hxy, self.z)
        w = self.w
        mass = (w[:, None, None, None] * w[:, None, None] * (self.dz[:, None] * w))[None] \
            * self.col(0.125 * self.dx * self.dy)
        ref = _reference(zp)
        ref = self.scatter(torch.stack([ref["rho0"], ref["theta0"], ref["dth"]]))
        self.r0, self.t0, self.dth = self.elements(ref)
        p = PHYS
        self.gam = p["c_p"] / (p["c_p"] - p["R_d"])
        self.p0 = p["p00"] * (p["R_d"] * self.r0 * self.t0 / p["p00"]) ** self.gam
        if case["terrain"]:
            zl = self.scatter(zs[None, :, None])[0]                    # (nc, np1^2, 1)
            zl = zl.reshape(self.nc, self.np1, self.np1, 1, 1)
            self.zs = zl
            self.gs = 1.0 / (1.0 - zl / case["H"])
            tf = (1.0 - self.z / case["H"])[self.kidx][None, None, None]
            sx = self.along(zl, 2) * self.col(2.0 / self.dx)
            sy = self.along(zl, 1) * self.col(2.0 / self.dy)
            self.ax, self.ay = -tf * self.gs * sx, -tf * self.gs * sy
            mass = mass / self.gs
            mh = (w[:, None] * w)[None] * (0.25 * self.dx * self.dy)[:, None, None] / self.gs[..., 0, 0]
            g = self.gather(torch.stack([mh * sx[..., 0, 0], mh * sy[..., 0, 0], mh])
                            .reshape(3, self.nc, -1, 1))[..., 0]
            n = torch.stack([-g[0] / g[2], -g[1] / g[2], torch.ones_like(g[2])])
            self.normal = n / n.norm(dim=0)
        self.mass = mass
        self.M = self.gather(self.from_elements(mass[None].contiguous()))
        return x, y, zp

    def dp(self, e):
        return self.p0 * torch.expm1(self.gam * (torch.log1p(e[0] / self.r0) + torch.log1p(e[4] / self.t0)))

    def rhs(self, q):
        """(5, n_h, nzn) tendency of a state of that shape."""
        p, e = PHYS, self.elements(self.scatter(q))
        rp, u, v, w, th = e
        rho = self.r0 + rp
        R = torch.empty_like(e)
        R[0] = -(self.grad(rho * u)[0] + self.grad(rho * v)[1] + self.grad(rho * w)[2])
        px, py, pz = self.grad(self.dp(e))
        adv = lambda g: u * g[0] + v * g[1] + w * g[2]
        gu, gv, gw = self.grad(u), self.grad(v), self.grad(w)
        R[1] = -adv(gu) - px / rho + p["f"] * v
        R[2] = -adv(gv) - py / rho - p["f"] * u
        R[3] = -adv(gw) - pz / rho - rp / rho * p["g"]
        R[4] = -adv(self.grad(th)) - w * self.dth
        if self.case["cs"]:
            sxy, sxz, syz = 0.5 * (gu[1] + gv[0]), 0.5 * (gu[2] + gw[0]), 0.5 * (gv[2] + gw[1])
            ss = gu[0] ** 2 + gv[1] ** 2 + gw[2] ** 2 + 2.0 * (sxy ** 2 + sxz ** 2 + syz ** 2)
            nu2 = 2.0 * self.col(self.case["cs"] * (self.dx + self.dy) / (2.0 * self.N)) ** 2 * torch.sqrt(2.0 * ss)
            div = lambda a, b: self.grad(a)[0] + self.grad(b)[1]
            R[1] += div(nu2 * gu[0], nu2 * sxy)
            R[2] += div(nu2 * sxy, nu2 * gv[1])
            R[3] += div(nu2 * sxz, nu2 * syz)
            zt = self.case["H"] - self.z
            layer = torch.sin(0.5 * math.pi * (1.0 - zt / 4000.0)) ** 2
            layer = torch.where(zt <= 4000.0, layer.clamp(0.0, 1.0), torch.zeros_like(zt))
            R -= layer[self.kidx] * e
        out = self.gather(self.from_elements(R * self.mass)) / self.M
        if self.zs is not None:
            dn = (out[1:4, :, 0] * self.normal).sum(0)
            out[1:4, :, 0] -= dn * self.normal
        else:
            out[3, :, 0] = 0.0
        out[3, :, -1] = 0.0
        return out

    def padded(self, q):
        out = torch.zeros(5, q.shape[1], self.ldz, dtype=torch.float64, device=DEV)
        out[:, :, :self.nzn] = q
        return out.reshape(-1)


def _logits(net, X):
    n = net.double()
    W1, b1, W2, b2, W3, b3 = n.split([1024, 64, 4096, 64, 192, 3])
    h1 = torch.tanh(X @ W1.view(64, 16).T + b1)
    h2 = torch.tanh(h1 @ W2.view(64, 64).T + b2)
    return h2 @ W3.view(3, 64).T + b3


def _exact_boundary(case, seed):
    M = _Plain(case)
    x, y, zp = M.setup()
    q, qp = (_state(case, seed, x, y, zp, -1500.0 * k) for k in range(2))
    e, ep = M.elements(M.scatter(q)), M.elements(M.scatter(qp))
    rp, u, v, w, th = e
    gu, gv, gw, gp, gt = (M.grad(a) for a in (u, v, w, M.dp(e), th))
    zeta, zetap = gv[0] - gu[1], M.grad(ep[2])[0] - M.grad(ep[1])[1]
    nodes = (1, 2, 4)
    top = lambda a: a.amax(dim=nodes)                              # (nc, layer)
    norm = lambda g: torch.sqrt(g[0] ** 2 + g[1] ** 2 + g[2] ** 2)
    zmax, umax = top(zeta.abs()), top(torch.hypot(u, v))
    # columns sharing a unique node
    h = M.h.reshape(-1)
    hs, order = torch.sort(h)
    cs, pairs = order // M.np1 ** 2, []
    for o in range(1, 9):
        same = (hs[o:] == hs[:-o]) & (hs[o:] >= 0)
        a, b = cs[:-o][same], cs[o:][same]
        pairs += [a * M.nc + b, b * M.nc + a]
    pairs = torch.unique(torch.cat(pairs))
    a, b = pairs // M.nc, pairs % M.nc
    a, b = a[a != b], b[a != b]
    near = [torch.zeros_like(zmax).index_reduce_(0, a, t[b], "amax") for t in (zmax, umax)]
    lvl = max(case["levels"], 1)
    thr = torch.tensor(THRESHOLDS[:lvl], dtype=torch.float64, device=DEV)
    cm, lev = top(zeta), M.lev[:, None]
    up = (lev < lvl) & (cm > thr[lev.clamp(max=lvl - 1)])
    down = ~up & (lev > 0) & (cm <= thr[(lev - 1).clamp(min=0)])
    f = [lev.double().expand_as(cm), zmax, zeta.mean(dim=nodes), umax, top(w.abs()), top(th),
         th.amin(dim=nodes), top(norm(gp)), top(norm(gt)), top((gu[0] + gv[1] + gw[2]).abs()),
         top(rp) - rp.amin(dim=nodes), near[0], near[1], umax - top(torch.hypot(ep[1], ep[2])),
         zmax - top(zetap.abs()), up.double() - down.double()]
    feat = (torch.stack(f, dim=-1) * torch.as_tensor(SCALE, device=DEV).double()).reshape(-1, 16)
    wind = torch.hypot(q[1], q[2]).max().reshape(1)
    return dict(plain=None, plain_col=None, wind=wind, feat=feat.reshape(-1), dem=None,
                logits=_logits(_network(seed).to(DEV), feat).reshape(-1), flags=None, flags_col=None)


def _exact_transfer(case, seed):
    A, B = _Plain(case), _Plain(case, case["shift"])
    x, y, zp, _ = _points(case, A.hxy, A.z)
    loc = A.scatter(_state(case, seed, x, y, zp)).reshape(5, A.nc, A.np1, A.np1, A.nzn)
    half = [_lagrange(A.x, 0.5 * (A.x + s)) for s in (-1.0, 1.0)]       # child values of a parent
    # 1-D projection of two children onto the parent: mass-weighted least squares
    V, W = torch.cat(half), torch.cat([A.w, A.w])
    proj = torch.linalg.solve(V.T @ (W[:, None] * V), (V * W[:, None]).T).split(A.np1, dim=1)
    def tensor(f, py, px):                                     # apply along j and i
        f = torch.tensordot(f, py, dims=([2], [1])).movedim(-1, 2)
        return torch.tensordot(f, px, dims=([3], [1])).movedim(-1, 3)
    ident = torch.eye(A.np1, dtype=torch.float64, device=DEV)
    top = int(max(A.lev.max(), B.lev.max()))
    def table(ids, l):
        g = torch.full((case["nx"] << l, case["ny"] << l), -1, dtype=torch.long, device=DEV)
        s = torch.nonzero(A.lev == l)[:, 0]
        g[A.ix[s], A.iy[s]] = s
        return g
    grids = [table(A, l) for l in range(top + 2)]
    new = torch.zeros(5, B.nc, B.np1, B.np1, B.nzn, dtype=torch.float64, device=DEV)
    merged = torch.zeros(B.nc, dtype=torch.bool, device=DEV)
    for l in range(top + 1):
        c = torch.nonzero(B.lev == l)[:, 0]
        ix, iy = B.ix[c], B.iy[c]
        same = grids[l][ix, iy]
        k = same >= 0
        new[:, c[k]] = tensor(loc[:, same[k]], ident, ident)
        if l > 0:
            par = grids[l - 1][ix // 2, iy // 2]
            for a in (0, 1):
                for b in (0, 1):
                    s = (par >= 0) & ~k & (ix % 2 == a) & (iy % 2 == b)
                    new[:, c[s]] = tensor(loc[:, par[s]], half[b], half[a])
            k = k | (par >= 0)
        m = ~k
        merged[c[m]] = True
        for a in (0, 1):
            for b in (0, 1):
                ch = grids[l + 1][2 * ix[m] + a, 2 * iy[m] + b]
                new[:, c[m]] += tensor(loc[:, ch], proj[b], proj[a])
    # nodes of kept or split columns take those columns' value, the others the
    # lumped-mass average of the merged ones
    wgt = (A.w[:, None] * A.w)[None] * (B.dx * B.dy)[:, None, None]
    def mean(sel):
        ok = (B.h.reshape(-1) >= 0) & sel[:, None].expand(-1, B.np1 ** 2).reshape(-1)
        hs, ws = B.h.reshape(-1)[ok], wgt.reshape(-1)[ok]
        num = torch.zeros(5, B.n_h, B.nzn, dtype=torch.float64, device=DEV)
        num.index_add_(1, hs, new.reshape(5, -1, B.nzn)[:, ok] * ws[None, :, None])
        den = torch.zeros(B.n_h, dtype=torch.float64, device=DEV).index_add_(0, hs, ws)
        return num / den.clamp(min=1e-300)[None, :, None], den > 0
    (kept, has), (avg, _) = mean(~merged), mean(merged)
    return B.padded(torch.where(has[None, :, None], kept, avg))


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        X, Y, idx = _samples(seed, case["batch"])
        rows = idx[0].long()
        net = _network(seed).to(DEV)
        w = net.double().clone().requires_grad_(True)
        loss = torch.nn.functional.cross_entropy(_logits(w, X[rows].double().to(DEV)),
                                                 Y[rows].long().to(DEV))
        loss.backward()
        g = w.grad
        step = 1e-3 * g / (g.abs() + 1e-8)
        return [g, loss.detach().reshape(1), net.double() - step, 0.1 * g, 0.001 * g * g]
    if kind == "boundary":
        return _exact_boundary(case, seed)
    if kind == "transfer":
        return _exact_transfer(case, seed)
    M = _Plain(case)
    q = _state(case, seed, *M.setup())
    dt = _time_step(case)
    if kind == "rhs":
        r = M.rhs(q)
        return [M.padded(r), M.padded(q + 0.25 * dt * r)]
    qs = q
    for a, b, c in RK3:
        qs = a * q + b * qs + c * dt * M.rhs(qs)
    return M.padded(qs)

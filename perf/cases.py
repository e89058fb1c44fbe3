"""Timed workloads: what a user of the library has it do, from the smallest call to the
largest run.

Most cases are whole jobs, as a program runs them (and as serve.run_plain_one does): a
context on one realization, its seed, its steps, then the per-cell results left on the
device and the tallies read back.  Nothing of a job can be kept between passes, since a
context's particles evolve; so every pass is a fresh realization from creation to
results.  The others are the kernel-level entry points on device arrays (the counting
sort, zero-dimensional reactors), the batched ensemble kept resident as a server keeps
it, and a restart from a checkpoint with the field and density queries.

Sizes are those of workloads.py (the 32^3 and 256^3 avalanches, the 64^3 and 256^3
streamers, the dense and the TSC streamer, the served 128^3 and reactor requests, the
batched realizations); step counts are shortened where a full run takes minutes.  Grids
of self-consistent cases have to coarsen by halving to at most 4096 cells, so "ragged"
ones are small odd multiples of powers of two.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2307_01797_amd import itokmc, serve, workloads

DEV = "cuda:0"
E_CHARGE = 1.602176634e-19
EPS0 = 8.8541878128e-12

# tallies of itokmc_diagnostics that are results (the others report on the solver or on
# the launches)
TALLIES = ("n_particles", "weight", "n_plus", "n_minus", "charge", "outflow_weight", "photons_emitted",
           "photons_absorbed", "photons_lost", "created", "removed_weight", "merged_cells", "step",
           "occupied_cells", "particle_steps", "ion_outflow_plus", "ion_outflow_minus")


def listed():
    return [
        # the smallest call: the sort of a few thousand particles inside a caller's loop,
        # through the form that allocates nothing
        dict(name="sort_small", kind="sort", n=3001, grid_x=32, grid_y=32, grid_z=32, fp64=True,
             noalloc=True, jitter=1.0),
        # one served zero-dimensional request: 4096 reactors, mid-range field and steps
        dict(name="reactor_request", kind="reactors", n=4096, E=4.5e6, X0=10, steps=275, dt=1e-12),
        # the reaction-algorithm comparison at full size (case a: 10 MV/m, one electron)
        dict(name="reactors_1e6", kind="reactors", n=1_000_000, E=1.0e7, X0=1, steps=50, dt=1e-12),
        # the plain avalanche at the size of the reference runs, all of its 200 steps, FP64
        dict(name="avalanche_32", kind="avalanche", n0=10_000, grid_x=32, grid_y=32, grid_z=32, dx=10e-6,
             E=1.0e7, sigma=50e-6, fp64=True, steps=200, dt=1e-12, merge=0, photons=False),
        # the avalanche at streamer scale: 5e7 electrons on 256^3, FP32
        dict(name="avalanche_256", kind="avalanche", n0=50_000_000, grid_x=256, grid_y=256, grid_z=256,
             dx=1e-3 / 256, E=1.0e7, sigma=150e-6, fp64=False, steps=10, dt=1e-12, merge=0, photons=False),
        # a batch of independent realizations run to completion on a resident ensemble
        dict(name="ensemble_32", kind="ensemble", realizations=32, steps=500, stop=1_000_000),
        # a restart: state from host memory, the field it stands in, the next time step and
        # the per-cell queries; ragged grid, FP64, a tight solver tolerance
        dict(name="restart_field", kind="restart", n=200_000, grid_x=72, grid_y=56, grid_z=88, dx=8e-6,
             tsc=False, fp64=True, V=18e3),
        # one served self-consistent request (128^3, no merging), the start of its 500 steps
        dict(name="poisson_128", kind="request", grid=128, E=7.0e6, n0=20_000, steps=60),
        # the precision study's streamer with recombination and mobile ions, FP64
        dict(name="streamer_64_fp64", kind="streamer", grid_x=64, grid_y=64, grid_z=64, dx=1e-3 / 64, V=18e3,
             peak=1e20, sigma=40e-6, centre_z=0.9, fp64=True, tsc=False, ions=True, recomb=True, steps=40),
        # the headline run
        dict(name="streamer_256", kind="streamer", grid_x=256, grid_y=256, grid_z=256, dx=1e-3 / 256, V=18e3,
             peak=1e20, sigma=40e-6, centre_z=0.9, fp64=False, tsc=False, ions=False, recomb=False, steps=20),
        # the higher-order shape on a ragged grid
        dict(name="streamer_tsc", kind="streamer", grid_x=176, grid_y=144, grid_z=208, dx=5e-6, V=18e3,
             peak=1e20, sigma=40e-6, centre_z=0.85, fp64=False, tsc=True, ions=False, recomb=False, steps=12),
        # the streamer near the particle cap
        dict(name="streamer_dense", kind="streamer", grid_x=256, grid_y=256, grid_z=256, dx=1e-3 / 256, V=18e3,
             peak=1e21, sigma=65e-6, centre_z=0.5, fp64=False, tsc=False, ions=False, recomb=False, steps=6),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _ragged(rng, target):
    """Three axis lengths m 2^p near target that coarsen by halving to at most 15^3 cells."""
    p = max(0, int(round(math.log2(target / 10.0))))
    lo, hi = 7, 15
    out = []
    for _ in range(3):
        m = rng.randint(lo, hi)
        out.append(min(256, max(4, m << p)))
    return out


def draw(rng):
    kind = rng.choice(["sort", "reactors", "avalanche", "avalanche", "ensemble", "restart", "request",
                       "streamer", "streamer", "streamer"])
    if kind == "sort":
        n = int(_log(rng, 500, 3e7))
        e = [rng.randint(16, 250) for _ in range(3)]
        small = n < 1_000_000 and e[0] * e[1] * e[2] < 6_000_000
        return dict(kind="sort", n=n, grid_x=e[0], grid_y=e[1], grid_z=e[2], fp64=rng.random() < 0.4,
                    noalloc=small and rng.random() < 0.5, jitter=round(rng.uniform(0.2, 4.0), 3))
    if kind == "reactors":
        n = int(_log(rng, 1000, 1.2e6))
        steps = rng.randint(50, 500 if n < 200_000 else 60)
        return dict(kind="reactors", n=n, E=round(_log(rng, 1.7e6, 1.2e7)), X0=int(_log(rng, 1, 100)),
                    steps=steps, dt=1e-12)
    if kind == "avalanche":
        n0 = int(_log(rng, 1000, 3e7))
        base = 24 if n0 < 100_000 else (72 if n0 < 2_000_000 else 160)
        e = [rng.randint(base, int(1.5 * base)) for _ in range(3)]
        dx = 4e-6
        return dict(kind="avalanche", n0=n0, grid_x=e[0], grid_y=e[1], grid_z=e[2], dx=dx,
                    E=round(_log(rng, 3e6, 1.2e7)), sigma=0.15 * min(e) * dx, fp64=rng.random() < 0.35,
                    steps=rng.randint(8, 120) if n0 < 1_000_000 else rng.randint(4, 12), dt=1e-12,
                    merge=rng.choice([0, 0, 32]), photons=rng.random() < 0.3)
    if kind == "ensemble":
        return dict(kind="ensemble", realizations=rng.randint(1, 40), steps=rng.randint(50, 400),
                    stop=500_000)
    if kind == "restart":
        g = _ragged(rng, rng.uniform(20, 100))
        return dict(kind="restart", n=int(_log(rng, 1000, 300_000)), grid_x=g[0], grid_y=g[1], grid_z=g[2],
                    dx=8e-6, tsc=rng.random() < 0.4, fp64=True, V=round(rng.uniform(5e3, 2e4)))
    if kind == "request":
        return dict(kind="request", grid=rng.choice([48, 64, 80, 96, 112, 128]), E=round(_log(rng, 3e6, 1.2e7)),
                    n0=int(_log(rng, 1000, 1e5)), steps=rng.randint(20, 80))
    big = rng.random() < 0.35
    g = _ragged(rng, rng.uniform(120, 250) if big else rng.uniform(28, 110))
    dx = round(_log(rng, 4e-6, 1.2e-5), 9)
    L = min(g) * dx
    fp64 = (not big) and rng.random() < 0.4
    return dict(kind="streamer", grid_x=g[0], grid_y=g[1], grid_z=g[2], dx=dx,
                V=round(1.8e7 * g[2] * dx), peak=round(_log(rng, 2e19, 2e20)), sigma=min(40e-6, 0.1 * L),
                centre_z=round(rng.uniform(0.5, 0.88), 3), fp64=fp64, tsc=rng.random() < 0.35,
                ions=rng.random() < 0.3, recomb=rng.random() < 0.3,
                steps=rng.randint(4, 12) if big else rng.randint(8, 40))


# ---- configurations ---------------------------------------------------------------------


def _grid(case):
    return (int(case["grid_x"]), int(case["grid_y"]), int(case["grid_z"]))


def _cfg(case, seed):
    """The descriptor of a whole-job case; the seed is the key of its random streams."""
    kind = case["kind"]
    if kind == "avalanche":
        g = _grid(case)
        c = workloads.preset("avalanche_32", grid=g, dx=case["dx"], E=(0.0, 0.0, float(case["E"])),
                             seed_n0=int(case["n0"]), seed_sigma=case["sigma"],
                             seed_centre=tuple(0.5 * a * case["dx"] for a in g), dt=case["dt"],
                             precision="fp64" if case["fp64"] else "fp32", n_ppc=int(case["merge"]),
                             steps=int(case["steps"]))
        if case["photons"]:
            c["coeffs"]["kgamma_ratio"] = 0.06
        rate = float(itokmc.rates(c, case["E"])[0])
        grown = case["n0"] * math.exp(min(6.0, 1.1 * rate * case["dt"] * case["steps"]))
        c["max_particles"] = int(1.5 * grown + 20 * math.sqrt(grown)) + 200_000
    elif kind == "request":
        n = int(case["grid"])
        L = n * 5e-6
        c = workloads.poisson_request(0, seed)
        c.update(grid=(n, n, n), V_anode=case["E"] * L, seed_n0=int(case["n0"]), steps=int(case["steps"]),
                 seed_centre=(L / 2, L / 2, L / 2), seed_sigma=0.156 * L)
    else:
        g = _grid(case)
        dx = case["dx"]
        c = workloads.preset("streamer_256", grid=g, dx=dx, V_anode=float(case["V"]), seed_peak=float(case["peak"]),
                             seed_sigma=case["sigma"],
                             seed_centre=(0.5 * g[0] * dx, 0.5 * g[1] * dx, case["centre_z"] * g[2] * dx),
                             precision="fp64" if case["fp64"] else "fp32", shape="tsc" if case["tsc"] else "cic",
                             steps=int(case["steps"]))
        if case["ions"]:
            c["coeffs"].update(workloads.IONS)
        if case["recomb"]:
            c["coeffs"].update(workloads.RECOMBINATION)
        c["max_particles"] = _seed_particles(case) * 2 + 2_000_000
    c["seed"] = int(seed) & 0x7FFFFFFF
    return c


def _seed_particles(case):
    """About how many computational particles the neutral seed makes (at most 64 a cell)."""
    peak = case["peak"] * case["dx"] ** 3
    s = case["sigma"] / case["dx"]
    r = np.linspace(0.0, 8.0 * s, 4001)
    lam = peak * np.exp(-r * r / (2 * s * s))
    return int(np.sum(np.minimum(64.0, lam) * 4 * math.pi * r * r) * (r[1] - r[0]))


# ---- the passes -------------------------------------------------------------------------


def _tallies(d):
    return np.array([d[k] for k in TALLIES] + list(d["fires"]), dtype=np.int64)


def _query(sim, sel, dtype, per=1):
    out = torch.empty(sim.ncell * per, dtype=dtype, device=sim.device)
    sim._check(itokmc.lib().itokmc_deposit(sim.h, sel, ctypes.c_void_p(out.data_ptr())))
    return out


def _state_out(sim, field):
    out = dict(weight=_query(sim, itokmc.Q_NGP_WEIGHT, torch.int32),
               plus=_query(sim, itokmc.Q_NPLUS, torch.int32),
               minus=_query(sim, itokmc.Q_NMINUS, torch.int32),
               gamma=_query(sim, itokmc.Q_NGAMMA, torch.int32),
               fires=_query(sim, itokmc.Q_FIRES, torch.int32, 3))
    if field:
        out["phi"] = _query(sim, itokmc.Q_PHI, torch.float64)
    else:
        out["density"] = _query(sim, itokmc.Q_CIC_DENSITY, torch.float64)
    return out


def _sort_inputs(case, seed):
    """Particles grouped by cell up to a displacement of `jitter` cells (what a push
    leaves), every 16th slot dead, in a plume over the middle of the grid."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    nx, ny, nz = _grid(case)
    n = int(case["n"])
    ft = torch.float64 if case["fp64"] else torch.float32
    p = torch.randn(n, 3, device=DEV, generator=g) * 0.15 + 0.5
    p = p.clamp(0.0, 0.999999) * torch.tensor([nx, ny, nz], device=DEV)
    old = p.long()
    key = old[:, 0] + nx * (old[:, 1] + ny * old[:, 2])
    p = p[torch.argsort(key)]
    p = p + torch.randn(n, 3, device=DEV, generator=g) * 0.1 * float(case["jitter"])
    i = p.floor().long()
    lim = torch.tensor([nx, ny, nz], device=DEV)
    ok = ((i >= 0) & (i < lim)).all(1)
    cell = torch.where(ok, i[:, 0] + nx * (i[:, 1] + ny * i[:, 2]), torch.zeros_like(i[:, 0]))
    w = (ok & (torch.rand(n, device=DEV, generator=g) > 1 / 16)).to(torch.int32)
    off = torch.rand(3, n, device=DEV, generator=g, dtype=ft)
    return [cell.to(torch.int32), off[0].clone(), off[1].clone(), off[2].clone(), w,
            torch.randperm(n, device=DEV, generator=g)]


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind == "sort":
        t = _sort_inputs(case, seed)
        nc = int(np.prod(_grid(case)))
        o = [torch.zeros_like(x) for x in t]
        start = torch.zeros(nc + 1, dtype=torch.int32, device=DEV)
        cnt = torch.zeros(1, dtype=torch.int32, device=DEV)
        st.update(t=t, o=o, start=start, cnt=cnt, ncell=nc)
        if not case["noalloc"]:
            st["ws"] = torch.empty(itokmc.lib().itokmc_sort_workspace_bytes(int(case["n"]), nc),
                                   dtype=torch.uint8, device=DEV)
    elif kind == "reactors":
        n = int(case["n"])
        cfg = dict(workloads.REACTOR_A, seed=int(seed) & 0x7FFFFFFF)
        st["sim"] = itokmc.Sim(cfg, device=DEV, max_particles=1024)
        X = torch.zeros(n, 4, dtype=torch.int64, device=DEV)
        X[:, 0] = int(case["X0"])
        k = torch.from_numpy(itokmc.rates(cfg, float(case["E"]))).to(DEV).expand(n, 5).contiguous()
        st.update(X0=X, X=X.clone(), k=k, ids=torch.arange(n, dtype=torch.int32, device=DEV),
                  fires=torch.zeros(n, 5, dtype=torch.int64, device=DEV))
    elif kind == "ensemble":
        cfgs = []
        for r in range(int(case["realizations"])):
            c = workloads.ensemble_realization(r, seed=int(seed) & 0x7FFFFFFF)
            c.update(steps=int(case["steps"]), stop_particles=int(case["stop"]))
            cfgs.append(c)
        st.update(cfgs=cfgs, ens=serve.ensemble_for(cfgs, device=DEV))
    elif kind == "restart":
        rng = np.random.default_rng(int(seed))
        g = _grid(case)
        n, nc = int(case["n"]), int(np.prod(g))
        xi = np.clip(rng.normal(0.5, 0.16, (n, 3)), 0.0, 0.999999) * np.array(g)
        ijk = np.floor(xi).astype(np.int64)
        cell = (ijk[:, 0] + g[0] * (ijk[:, 1] + g[1] * ijk[:, 2])).astype(np.uint32)
        cfg = workloads.preset("streamer_256", grid=g, dx=case["dx"], V_anode=float(case["V"]), precision="fp64",
                               shape="tsc" if case["tsc"] else "cic", gmg_rtol=1e-12, max_particles=2 * n + 1000)
        w = rng.integers(1, 40, n).astype(np.uint32)
        plus = np.bincount(cell, weights=w, minlength=nc).astype(np.uint32) + (rng.random(nc) < 0.05).astype(np.uint32)
        st.update(cfg=cfg, cell=cell, off=np.minimum(xi - ijk, 1 - 2.0 ** -53), w=w, ids=np.arange(n, dtype=np.uint64),
                  plus=plus, minus=(rng.random(nc) < 0.02).astype(np.uint32),
                  rule=dict(dt_max=2e-12, c_drift=0.5, c_ion=0.1))
    else:
        st["cfg"] = _cfg(case, seed)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "sort":
        p = [ctypes.c_void_p(x.data_ptr()) for x in st["t"] + st["o"] + [st["start"], st["cnt"]]]
        prec = itokmc.FP64 if case["fp64"] else itokmc.FP32
        s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        L = itokmc.lib()
        if case["noalloc"]:
            rc = L.itokmc_sort_by_cell_noalloc(prec, int(case["n"]), st["ncell"], *p, s)
        else:
            rc = L.itokmc_sort_by_cell(prec, int(case["n"]), st["ncell"], *p, ctypes.c_void_p(st["ws"].data_ptr()),
                                       st["ws"].numel(), s)
        if rc:
            raise itokmc.ItokmcError(rc, "sort")
        # the order inside a cell is unspecified: offsets and ids are permuted from call to call
        return dict(start=st["start"], n=st["cnt"], cell=st["o"][0], w=st["o"][4])
    if kind == "reactors":
        st["X"].copy_(st["X0"])
        st["sim"].kmc_run_device(st["ids"], st["X"], st["k"], float(case["dt"]), 0, int(case["steps"]), st["fires"])
        return dict(X=st["X"], fires=st["fires"])
    if kind == "ensemble":
        r = serve.run_batched(st["cfgs"], ens=st["ens"], device=DEV)["results"]
        return dict(tallies=np.stack([_tallies(d) for d in r]), state=np.array([d["state"] for d in r]))
    if kind == "restart":
        sim = itokmc.Sim(st["cfg"], device=DEV)
        try:
            sim.set_particles(st["cell"], st["off"], st["w"], st["ids"])
            sim.set_counts("plus", st["plus"])
            sim.set_counts("minus", st["minus"])
            dt, Emax = sim.stable_dt(st["rule"])
            out = dict(next=np.array([dt, Emax]))
            for k, q in (("phi", itokmc.Q_PHI), ("ex", itokmc.Q_EX), ("ey", itokmc.Q_EY), ("ez", itokmc.Q_EZ),
                         ("density", itokmc.Q_CIC_DENSITY), ("rho", itokmc.Q_RHO)):
                out[k] = _query(sim, q, torch.float64)
            return out
        finally:
            sim.close()
    cfg = st["cfg"]
    sim = itokmc.Sim(cfg, device=DEV)
    try:
        sim.seed()
        if kind == "request":
            sim.step_until(cfg["steps"], cfg["stop_particles"])
        else:
            sim.step(cfg["steps"])
        out = _state_out(sim, cfg.get("field") == "poisson")
        out["tallies"] = _tallies(sim.diagnostics())
        return out
    finally:
        sim.close()


# ---- what a pass cannot do without ------------------------------------------------------


def work(case):
    """Bytes: a step reads and writes each particle's state once (28 B in FP32, 40 in FP64;
    the number of particles is that of the seed) and, self-consistent, the potential, the
    coefficient and the charge of each cell; flops: some hundred for each particle."""
    kind = case["kind"]
    if kind == "sort":
        n, s = case["n"], 40 if case["fp64"] else 28
        return dict(bytes=2 * n * s + 4 * int(np.prod(_grid(case))), flops=2 * n)
    if kind == "reactors":
        return dict(bytes=case["n"] * (64 + 44 + 40), flops=100 * case["n"] * case["steps"])
    if kind == "ensemble":
        n = case["realizations"] * 21_500
        return dict(bytes=56 * n * case["steps"], flops=150 * n * case["steps"])
    if kind == "restart":
        nc, n = int(np.prod(_grid(case))), case["n"]
        return dict(bytes=nc * (8 + 48 + 8) + 44 * n, flops=200 * nc + 100 * n)
    s = 40 if case.get("fp64") else 28
    if kind == "avalanche":
        n, nc = case["n0"], 0
    elif kind == "request":
        n, nc = case["n0"], int(case["grid"]) ** 3
    else:
        n, nc = _seed_particles(case), int(np.prod(_grid(case)))
    return dict(bytes=case["steps"] * (2 * s * n + 32 * nc), flops=case["steps"] * (200 * n + 200 * nc))


# ---- values in 64 bits ------------------------------------------------------------------


def _axis(c, t, n, tsc):
    """Node indices and weights of one axis: c + t in cells, clouds folded into the walls."""
    x = c + t
    if tsc:
        j = np.floor(x).astype(np.int64)
        d = x - j - 0.5
        return [(np.clip(j - 1, 0, n - 1), 0.5 * (0.5 - d) ** 2), (j, 0.75 - d * d),
                (np.clip(j + 1, 0, n - 1), 0.5 * (0.5 + d) ** 2)]
    lo = np.floor(x - 0.5)
    f = x - 0.5 - lo
    lo = lo.astype(np.int64)
    return [(np.clip(lo, 0, n - 1), 1.0 - f), (np.clip(lo + 1, 0, n - 1), f)]


def _spread(ijk, t, q, g, tsc):
    out = np.zeros(int(np.prod(g)))
    ax = [_axis(ijk[:, a].astype(np.float64), t[:, a], g[a], tsc) for a in range(3)]
    for ix, wx in ax[0]:
        for iy, wy in ax[1]:
            for iz, wz in ax[2]:
                out += np.bincount(ix + g[0] * (iy + g[1] * iz), weights=q * wx * wy * wz, minlength=len(out))
    return out


def exact(case, seed):
    """The restart's density, charge, potential and field: the charge deposited with the
    shape's weights, the 7-point system (Neumann in x and y, potentials 0 and V on the z
    faces) diagonalised by its cosine and sine modes.  The runs that evolve have no value
    in 64 bits that plain arithmetic gives; the sort and the reactors give whole numbers."""
    if case["kind"] != "restart":
        return None
    st = _restart_host(case, seed)
    g, dx, V = st["g"], case["dx"], float(case["V"])
    dV = dx ** 3
    ne = _spread(st["ijk"], st["off"], st["w"].astype(np.float64), g, case["tsc"])
    ions = st["plus"].astype(np.float64) - st["minus"]
    if case["tsc"]:
        c = np.arange(len(ions))
        ijk = np.stack([c % g[0], (c // g[0]) % g[1], c // (g[0] * g[1])], 1)
        ions = _spread(ijk, np.full((len(c), 3), 0.5), ions, g, True)
    nx, ny, nz = g
    b = ((ions - ne) * (dx * dx * E_CHARGE / (EPS0 * dV))).reshape(nz, ny, nx)
    b[-1] += 2.0 * V

    def cos_modes(n):
        k, i = np.arange(n)[:, None], np.arange(n)[None, :]
        m = np.cos(math.pi * k * (i + 0.5) / n) * math.sqrt(2.0 / n)
        m[0] = math.sqrt(1.0 / n)
        return m, 4 * np.sin(math.pi * np.arange(n) / (2 * n)) ** 2

    def sin_modes(n):
        k, i = np.arange(1, n + 1)[:, None], np.arange(n)[None, :]
        m = np.sin(math.pi * k * (i + 0.5) / n) * math.sqrt(2.0 / n)
        m[-1] = m[-1] / math.sqrt(2.0)
        return m, 4 * np.sin(math.pi * np.arange(1, n + 1) / (2 * n)) ** 2

    Cx, lx = cos_modes(nx)
    Cy, ly = cos_modes(ny)
    Sz, lz = sin_modes(nz)
    h = np.einsum("zyx,ax->zya", b, Cx, optimize=True)
    h = np.einsum("zya,by->zba", h, Cy, optimize=True)
    h = np.einsum("zba,cz->cba", h, Sz, optimize=True)
    h /= lz[:, None, None] + ly[None, :, None] + lx[None, None, :]
    h = np.einsum("cba,cz->zba", h, Sz, optimize=True)
    h = np.einsum("zba,by->zya", h, Cy, optimize=True)
    phi = np.einsum("zya,ax->zyx", h, Cx, optimize=True)
    x = np.concatenate([phi[:, :, :1], phi, phi[:, :, -1:]], 2)
    y = np.concatenate([phi[:, :1], phi, phi[:, -1:]], 1)
    z = np.concatenate([-phi[:1], phi, 2 * V - phi[-1:]], 0)
    ex = -(x[:, :, 2:] - x[:, :, :-2]) / (2 * dx)
    ey = -(y[:, 2:] - y[:, :-2]) / (2 * dx)
    ez = -(z[2:] - z[:-2]) / (2 * dx)
    Em = float(np.sqrt(ex * ex + ey * ey + ez * ez).max())
    a = st["coeffs"]
    v = a["mu_a"] * (max(Em, a["E_floor"]) / a["mu_E0"]) ** a["mu_b"] * Em
    nu = a["alpha_A"] * math.exp(-a["alpha_B"] / Em) * v
    r = st["rule"]
    dt = min(r["dt_max"], r["c_drift"] * dx / v, r["c_ion"] / nu if nu > 0 else math.inf)
    t = lambda m: torch.from_numpy(np.ascontiguousarray(m).reshape(-1))  # noqa: E731
    return dict(next=np.array([dt, Em]), phi=t(phi), ex=t(ex), ey=t(ey), ez=t(ez), density=t(ne / dV),
                rho=t(E_CHARGE * (ions - ne) / dV))


def _restart_host(case, seed):
    st = prepare(case, seed)
    g = _grid(case)
    c = st["cell"].astype(np.int64)
    return dict(g=g, ijk=np.stack([c % g[0], (c // g[0]) % g[1], c // (g[0] * g[1])], 1), off=st["off"], w=st["w"],
                plus=st["plus"], minus=st["minus"], coeffs=st["cfg"]["coeffs"], rule=st["rule"])

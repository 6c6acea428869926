"""Timed workloads of the ion-pack library, through its public binding.

listed() names the workloads, draw(rng) gives more of the same ranges,
prepare(case, seed) builds what a program holds before the call, run(state)
is one pass, work(case) the bytes and operations a pass cannot do without and
exact(case, seed) the outputs in plain 64-bit numpy where they have such a
value.  Four kinds:

  deposit  the stand-alone charge deposit of device tensors
  field    one space-charge update of a context and the read-back of its grids
  run      a stretch of steps of one simulation and the read-back of what its
           program looks at: the packs (populations up to some 1e5), or the
           tallies and space-charge grids (production populations, whose packs
           stay on the GPU)
  serve    a batch of design queries through the serving loop

A run with "replay" starts each pass from the same pack snapshot, as a
parameter study does; without it the population goes on from the last pass
(no packs are emitted then, and the passes cover a few millimetres).
"""
import math

import numpy as np
import torch

from paper_2609_31258_amd import mucite, synth

# The grid spacing of every workload (m) and the charge that a population
# carries in all, in real ions: 1e6 packs at the 256x1024 workload's weight.
H = 5e-5
REAL_IONS = 1.25e4

RUN = dict(kind="run", nr=128, nz=512, n=10_000, steps=100, fp32=False, fp32_tables=False, species=1, mass=500.0,
           charge=1, p0=1e5, p1=200.0, r_in=0.0, z_hi=3e-3, dt=1e-9, sc_every=0, mask=False, langevin=False,
           adaptive=False, sort_every=0, emit=0, replay=True, packs=True)


def _run(name, **changes):
    return {**RUN, **changes, "name": name}


def listed():
    return [
        # the charge of a small population, in a loop of a caller's own: launches and latency
        dict(name="deposit_small", kind="deposit", nr=128, nz=512, n=10_007, noalloc=False, spread=False),
        # a production population in the source region, where few cells share all of it
        dict(name="deposit_1e6", kind="deposit", nr=256, nz=1024, n=1_000_000, noalloc=False, spread=False),
        # one space-charge solve on the paper's 201x651 mesh, and its grids read back
        dict(name="field_201x651", kind="field", nr=201, nz=651, n=50_000),
        # the 128x512 workload: a small FP64 run at 1e5 Pa, tens of collisions per step
        _run("fp64_1e4"),
        # its low-pressure variant: few collisions, packs transmitted and lost on the way
        _run("fp64_lowp_1e4", steps=400, p0=1000.0, p1=20.0, r_in=2.5e-4, z_hi=0.0, dt=5e-9),
        # a design query's size in the precision form, ragged everywhere: continuous
        # emission, masked space charge on the paper's mesh
        _run("fp32_masked_30011", nr=201, nz=651, n=30_011, fp32=True, mass=2000.0, charge=3, dt=0.5e-9, sc_every=10,
             mask=True, emit=50),
        # the 256x1024 space-charge workload at its full population, in each form
        _run("fp64_1e6", nr=256, nz=1024, n=1_000_000, mass=5000.0, charge=5, dt=0.5e-9, sc_every=10, sort_every=100,
             replay=False, packs=False),
        _run("fp32_1e6", nr=256, nz=1024, n=1_000_000, fp32=True, mass=5000.0, charge=5, dt=0.5e-9, sc_every=10,
             sort_every=100, replay=False, packs=False),
        _run("hybrid_1e6", nr=256, nz=1024, n=1_000_000, steps=500, fp32=True, mass=5000.0, charge=5, dt=0.5e-9,
             sc_every=10, langevin=True, sort_every=100, replay=False, packs=False),
        # the large workload's ten species and cadences on a grid an eighth of its size
        _run("species10_8e5", nr=512, nz=2048, n=800_000, steps=60, fp32=True, species=10, dt=0.25e-9, sc_every=5,
             sort_every=20, replay=False, packs=False),
        # Eq. 1 steps on the Langevin branch, a mid-sized population with its packs read back
        _run("adaptive_1e5", nr=256, nz=1024, n=100_003, steps=200, fp32=True, mass=5000.0, charge=5, dt=5e-9,
             sc_every=10, langevin=True, adaptive=True),
        # a dozen design queries at once
        dict(name="serve_12", kind="serve", nr=256, nz=1024, queries=12, steps=100, n_lo=1000, n_hi=300_000,
             fp32=True),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["deposit", "deposit", "field", "run", "run", "run", "run", "serve"])
    nr, nz = rng.randint(100, 256), rng.randint(300, 1024)
    if kind == "deposit":
        return dict(kind=kind, nr=nr, nz=nz, n=int(_log(rng, 1000, 1_000_000)), noalloc=rng.random() < 0.5,
                    spread=rng.random() < 0.5)
    if kind == "field":
        return dict(kind=kind, nr=nr, nz=nz, n=int(_log(rng, 1000, 200_000)))
    if kind == "serve":
        return dict(kind=kind, nr=nr, nz=nz, queries=rng.randint(2, 12), steps=rng.randint(40, 100), n_lo=1000,
                    n_hi=rng.randint(20_000, 300_000), fp32=rng.random() < 0.75)
    c = dict(RUN, nr=nr, nz=nz, n=int(_log(rng, 500, 200_000)), fp32=rng.random() < 0.5, dt=0.5e-9,
             species=rng.choice([1, 1, 1, 4]), mass=float(int(_log(rng, 200, 20_000))), charge=rng.randint(1, 10))
    c["fp32_tables"] = c["fp32"] and rng.random() < 0.25
    if rng.random() < 0.4:  # rarefied, along the whole grid
        c.update(p0=_log(rng, 500, 5000), p1=20.0, r_in=2.5e-4, z_hi=0.0, dt=2e-9)
    if rng.random() < 0.5:
        c.update(sc_every=rng.randint(5, 20), mask=rng.random() < 0.5)
    c["langevin"] = rng.random() < 0.3
    c["adaptive"] = rng.random() < 0.15
    c["emit"] = rng.choice([0, 0, 25])
    c["sort_every"] = rng.choice([0, 0, 50])
    c["packs"] = c["sort_every"] == 0  # a sort drops the packs that have ended: the count varies
    c["steps"] = max(10, min(300, int(4e7 / c["n"])))
    # no more than the collisions of the largest listed case
    most = work(next(k for k in listed() if k["name"] == "fp64_1e6"))["flops"]
    while c["steps"] > 2 and work(c)["flops"] > most:
        c["steps"] //= 2
    return c


# ---------------------------------------------------------------------------
# prepare
# ---------------------------------------------------------------------------
def _fields(c):
    return synth.ring_fields(c["nr"], c["nz"], H, p0=c.get("p0", 1e5), p1=c.get("p1", 200.0),
                             r_in=c.get("r_in", 0.0) or None)


def _ions(c):
    if c["species"] > 1:
        return synth.config_c5_species(c["species"])
    m = c["mass"]
    return [synth.Ion(m, c["charge"], 200e-20 * (m / 500.0) ** (2.0 / 3.0), max(3, round(0.3 * m)), act_kind=1,
                      act_p1=100e3, act_p2=-80.0)]


def _operating(c, grid):
    return synth.Operating(dt=c["dt"], v_rf=100.0, f_rf=1e6, z_det=grid.L, r_det=grid.R, sc_on=int(c["sc_every"] > 0),
                           sc_every=max(1, c["sc_every"]), sc_mask=int(c["mask"]), langevin_on=int(c["langevin"]),
                           adaptive=int(c["adaptive"]), lv_dt_max=2e-9, sort_every=c["sort_every"],
                           exit_bin_dt=1e-7, n_exit_bins=1000)


def _snapshot(c, f, ions, seed):
    """Packs of a run under way: thermal about the gas flow, internally at 300-1500 K, in the source region
    (z_hi) or along the whole grid (z_hi = 0)."""
    n = c["n"]
    s = synth.c5_post_ramp_snapshot(f, ions, [REAL_IONS / n] * len(ions), n, seed)
    if not c["z_hi"]:
        s["z"] = np.random.default_rng(seed + 2).uniform(0.0, 0.95 * f.grid.L, n)
    return s


def _prepare_run(c, seed):
    f, ions = _fields(c), _ions(c)
    sim = mucite.Sim(seed=seed, pack_capacity=c["n"] + c["steps"] * c["emit"], precision=int(c["fp32"]),
                     fp32_tables=c["fp32_tables"])
    sources = [synth.Source(kind=1, ion=0, current_a=10e-9, packs_per_step=c["emit"], n_total=1 << 40, sigma_r=1e-4,
                            r_trunc=3e-4)] if c["emit"] else []
    sim.setup(f, ions, sources, _operating(c, f.grid))
    snap = _snapshot(c, f, ions, seed)
    snap["id"] += 1 << 50  # apart from the ids that the source gives
    sim.write_packs(snap)
    return dict(case=c, sim=sim, snap=snap)


def _field_case(c):
    return {**RUN, **c, "sc_every": 1}


def _charge_quanta(c, seed):
    rng = np.random.default_rng(seed)
    n, g = c["n"], synth.Grid(c["nr"], c["nz"], H, H)
    r = (0.9 * g.R if c["spread"] else 3e-4) * np.sqrt(rng.uniform(0, 1, n))
    ph = rng.uniform(0, 2 * math.pi, n)
    z = rng.uniform(0, 0.95 * g.L if c["spread"] else 3e-3, n)
    q = np.rint(5 * REAL_IONS / n * rng.uniform(0.5, 1.5, n) * 2.0**32).astype(np.int64)
    status = (rng.uniform(0, 1, n) < 0.03).astype(np.int32)  # a few have ended
    return g, r * np.cos(ph), r * np.sin(ph), z, q, status


def prepare(case, seed):
    c = case
    if c["kind"] == "deposit":
        g, *packs = _charge_quanta(c, seed)
        return dict(case=c, grid=g, packs=[torch.from_numpy(a).cuda() for a in packs],
                    out=torch.zeros(g.nr * g.nz, dtype=torch.int64, device="cuda"))
    if c["kind"] == "field":
        return dict(_prepare_run(_field_case(c), seed), case=c)
    if c["kind"] == "run":
        return _prepare_run(c, seed)
    f = _fields(c)
    queries = []
    for q in synth.serving_queries(c["queries"], seed=seed, pack_lo=c["n_lo"], pack_hi=c["n_hi"]):
        ion = synth.Ion(q["mass_da"], q["charge_z"], q["ccs_m2"], max(3, q["n_atoms"]), act_kind=1, act_p1=100e3,
                        act_p2=-80.0)
        src = synth.Source(kind=1, current_a=q["current_a"], n_total=q["n_packs"], sigma_r=1e-4, r_trunc=3e-4,
                           packs_per_step=max(1, round(q["n_packs"] / (c["steps"] // 2))))
        op = synth.Operating(dt=0.5e-9, v_rf=q["v_rf"], f_rf=1e6, v_off=q["v_off"], sc_on=1, sc_every=10,
                             z_det=f.grid.L, r_det=f.grid.R, exit_bin_dt=1e-7, n_exit_bins=100, sample_every=25,
                             sample_stride=1000)
        queries.append((ion, src, op, q["seed"]))
    server = mucite.Server(f, hbm_budget=8 << 30, precision=int(c["fp32"]), max_resident=16)
    return dict(case=c, server=server, queries=queries)


# ---------------------------------------------------------------------------
# run
# ---------------------------------------------------------------------------
def run(state):
    c = state["case"]
    if c["kind"] == "deposit":
        mucite.deposit_cic(*state["packs"], state["grid"], state["out"], noalloc=c["noalloc"])
        return state["out"]
    if c["kind"] == "serve":
        return _serve(state)
    sim, out = state["sim"], {}
    if c["kind"] == "field":
        sim.pic_update()
    else:
        if c["replay"]:
            sim.write_packs(state["snap"])
        sim.step(c["steps"])
        out["tallies"] = sim.read_tallies()
        if c["packs"]:
            out["packs"] = sim.read_packs()
    if c["kind"] == "field" or c["sc_every"]:
        out["charge"] = sim.read_charge()
        out["phi"], out["er"], out["ez"] = sim.read_sc()
    return out


SAMPLES = 2000  # records that a query keeps at most (its packs / 1000, every 25 steps)


def _serve(state):
    server, steps = state["server"], state["case"]["steps"]
    ids = [server.submit(ion, src, op, n_steps=steps, seed=seed, exit_capacity=1000, sample_capacity=SAMPLES)
           for ion, src, op, seed in state["queries"]]
    results = [server.wait(i) for i in ids]
    for i in ids:
        server.release(i)
    out = {k: np.stack([np.asarray(r["tallies"][k]) for r in results]) for k in results[0]["tallies"]}
    # (the records of a query come in no order of their own)
    samples = [r["samples"][np.lexsort((r["samples"]["id"], r["samples"]["step"]))] for r in results]
    for k in ("id", "step", "x", "y", "z", "vx", "vy", "vz", "ke_ev", "t_eff", "h", "w"):
        out["sample_" + k] = np.stack([np.pad(a[k], (0, SAMPLES - len(a))) for a in samples])
    return out


# ---------------------------------------------------------------------------
# work: operations of the method per pack-step and per candidate collision
# (one per add, multiply, compare, integer half product and elementary
# function), each input read once and each output written once per pass.
# ---------------------------------------------------------------------------
def _candidates(mass, ccs, p, dt):
    """Candidate collisions of a pack in a step: n sigma (s + abar) dt at 300 K nitrogen."""
    s = 1.6 * math.sqrt(synth.K_B * 300.0 / (mass * synth.DALTON))
    return p / (synth.K_B * 300.0) * ccs * (s + 476.0) * dt


def _run_ops(c):
    length = (c["nz"] - 1) * H
    z = 0.5 * (c["z_hi"] or 0.95 * length)
    p = c["p0"] * (c["p1"] / c["p0"]) ** (z / length)
    if c["langevin"] and p > 2e4:
        return 600.0  # the Langevin branch: no candidates
    cand = [min(0.1, _candidates(i.mass_da, i.ccs_m2, p, c["dt"])) if c["adaptive"]
            else _candidates(i.mass_da, i.ccs_m2, p, c["dt"]) for i in _ions(c)]
    return 567.0 + 430.0 * sum(cand) / len(cand)


def _update_ops(nr, nz):
    """Two sine transforms per row and one tridiagonal system per mode."""
    return nr * nz * (2 * 2.5 * math.log2(2 * nz) + 8)


def work(case):
    c = case
    nn = c["nr"] * c["nz"]
    if c["kind"] == "deposit":
        return {"bytes": 36.0 * c["n"] + 8.0 * nn, "flops": 40.0 * c["n"]}
    if c["kind"] == "field":
        return {"bytes": 36.0 * c["n"] + 32.0 * nn, "flops": 40.0 * c["n"] + _update_ops(c["nr"], c["nz"])}
    if c["kind"] == "serve":
        n = (c["n_hi"] - c["n_lo"]) / math.log(c["n_hi"] / c["n_lo"]) * c["queries"]  # mean of a log-uniform count
        cand = _candidates(3000.0, 200e-20 * 6.0 ** (2.0 / 3.0), 1e5, 0.5e-9)
        return {"bytes": 80.0 * n + c["queries"] * 8.0 * nn,
                "flops": 0.75 * n * c["steps"] * (567.0 + 430.0 * cand)
                + c["queries"] * c["steps"] / 10 * _update_ops(c["nr"], c["nz"])}
    updates = c["steps"] // c["sc_every"] if c["sc_every"] else 0
    state = 2.0 * (80 if c["fp32"] else 96) * c["n"]
    table = nn * (64.0 if not c["fp32"] else 32.0 if c["fp32_tables"] else 16.0)
    return {"bytes": state + table + (32.0 * nn if c["sc_every"] else 0.0) + 8.0 * nn,
            "flops": c["n"] * c["steps"] * _run_ops(c) + updates * _update_ops(c["nr"], c["nz"])}


# ---------------------------------------------------------------------------
# exact: the deposited charge is whole numbers and the solve has a value in 64
# bits.  A run is a chain of random accept-or-reject decisions, each of which
# depends on all before; following it in numpy takes minutes (1e6 and more
# pack-steps of some hundred operations times up to a hundred candidates).
# ---------------------------------------------------------------------------
def _deposit(x, y, z, q, active, nr, nz):
    grid = np.zeros(nr * nz, np.int64)
    x, y, z, q = x[active], y[active], z[active], q[active]
    ur, uz = np.sqrt(x * x + y * y) * (1.0 / H), z * (1.0 / H)
    i, j = np.minimum(np.floor(ur), nr - 2), np.clip(np.floor(uz), 0, nz - 2)
    f, g = np.minimum(ur - i, 1.0), np.clip(uz - j, 0.0, 1.0)
    inner = np.rint(q * (1.0 - f)).astype(np.int64)
    k = j.astype(np.int64) * nr + i.astype(np.int64)
    for part, o in ((inner, 0), (q - inner, 1)):
        low = np.rint(part * (1.0 - g)).astype(np.int64)
        np.add.at(grid, k + o, low)
        np.add.at(grid, k + o + nr, part - low)
    return grid


def _sine(a):
    """Unscaled DST-I along the last axis, by the FFT of the odd extension."""
    m = a.shape[-1]
    odd = np.zeros(a.shape[:-1] + (2 * (m + 1),))
    odd[..., 1:m + 1] = a
    odd[..., m + 2:] = -a[..., ::-1]
    return -0.5 * np.fft.rfft(odd, axis=-1).imag[..., 1:m + 1]


def _potential(charge, nr, nz):
    """Finite-volume cylindrical Poisson equation, zero at both ends and at r = R: sine modes along z, Thomas sweeps
    along r."""
    eps0, m, nu = 8.8541878188e-12, nz - 2, nr - 1
    i = np.arange(nu)
    volume = np.where(i == 0, math.pi * (0.5 * H) ** 2 * H, 2 * math.pi * (i * H) * H * H)
    b = -charge.reshape(nz, nr)[1:-1, :-1].T * (synth.E_CHARGE * 2.0**-32) / (volume * eps0)[:, None]
    d = _sine(b) * (2.0 / (nz - 1))
    lam = -(4.0 / H**2) * np.sin(math.pi * np.arange(1, m + 1) / (2.0 * (nz - 1))) ** 2
    r = np.maximum(i, 1) * H
    lo = np.where(i == 0, 0.0, (r - 0.5 * H) / (r * H * H))
    up = np.where(i == 0, 4.0 / H**2, (r + 0.5 * H) / (r * H * H))
    cp = np.zeros((nu, m))
    for k in range(nu):
        den = -(lo[k] + up[k]) + lam - (lo[k] * cp[k - 1] if k else 0.0)
        cp[k] = up[k] / den
        d[k] = (d[k] - (lo[k] * d[k - 1] if k else 0.0)) / den
    for k in range(nu - 2, -1, -1):
        d[k] -= cp[k] * d[k + 1]
    phi = np.zeros((nz, nr))
    phi[1:-1, :-1] = _sine(d).T
    return phi


def _field_of(phi):
    er, ez = np.zeros_like(phi), np.zeros_like(phi)
    er[:, 1:-1] = -(phi[:, 2:] - phi[:, :-2]) / (2 * H)
    er[:, -1] = -(phi[:, -1] - phi[:, -2]) / H
    ez[1:-1] = -(phi[2:] - phi[:-2]) / (2 * H)
    ez[0], ez[-1] = -(phi[1] - phi[0]) / H, -(phi[-1] - phi[-2]) / H
    return er, ez


def exact(case, seed):
    c = case
    if c["kind"] == "deposit":
        g, x, y, z, q, status = _charge_quanta(c, seed)
        return _deposit(x, y, z, q, status == 0, g.nr, g.nz)
    if c["kind"] != "field":
        return None
    full = _field_case(c)
    f, ions = _fields(full), _ions(full)
    s = _snapshot(full, f, ions, seed)
    q = np.rint(s["w"] * ions[0].charge_z * 2.0**32).astype(np.int64)
    charge = _deposit(s["x"], s["y"], s["z"], q, slice(None), c["nr"], c["nz"])
    phi = _potential(charge, c["nr"], c["nz"])
    er, ez = _field_of(phi)
    return {"charge": charge.reshape(c["nz"], c["nr"]), "phi": phi, "er": er, "ez": ez}

"""The stretch kernel (several steps per launch, 1 to 16 lanes per pack)
against one launch of the step kernel per step, bit for bit: a population of
140,000 packs stepped one step at a time takes the step kernel, stepped at
once the stretch kernel with one lane per pack, and subsets of it the stretch
kernel with 2 to 16 lanes (a pack's result depends on its id, state and step
alone while there is no space charge)."""
import sys

import numpy as np
import pytest

from paper_2609_31258_amd import synth

pytestmark = pytest.mark.gpu

STATE = ("x", "y", "z", "vx", "vy", "vz", "e_int", "h", "status")
INTS = ("class_n", "class_w", "n_cand", "n_coll", "n_cap", "n_clamp", "pack_steps", "n_langevin", "n_exchange",
        "exit_bins", "loss_map", "hist_ke", "hist_teff", "hist_r", "act_hist_ke", "act_hist_teff", "emitted_n",
        "emitted_w")
N = 140_000


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _scenario(name):
    """(fields, ions, sources, operating point, snapshot, steps)"""
    srcs = []
    if name == "exits":  # every terminal class, and more steps than one launch takes
        f, ions, _, op, _ = synth.config_c1x()
        rng = np.random.default_rng(5)
        snap = synth.pack_snapshot(N, f, seed=5, r_hi=9e-4, v_sigma=400.0)
        snap["z"] = np.where(rng.uniform(size=N) < 0.5, rng.uniform(25.0e-3, f.grid.L, N), rng.uniform(0, 23e-3, N))
        return f, ions, srcs, op, snap, 41
    f, ions, _, op, _ = synth.config_c1()
    snap = synth.pack_snapshot(N, f, seed=6, z_hi=4e-3, r_hi=5e-4, v_sigma=60.0)
    if name == "species":  # with emission: a fixed rate and the current accumulator
        ions = synth.config_c5_species(3)
        snap["tag"] = (np.arange(N) % 3).astype(np.int32)
        srcs = [synth.Source(kind=1, ion=1, current_a=1e-9, packs_per_step=37, n_total=300),
                synth.Source(kind=2, ion=2, current_a=2e-9, weight=0.31, n_total=10_000, step_start=2)]
        snap["id"] += 1 << 50
    elif name == "sorted":  # blocks from the last slot down (the last species collides most)
        ions = synth.config_c5_species(3)
        snap["tag"] = (np.arange(N) % 3).astype(np.int32)
        op.sort_every = 2
    elif name == "window":
        op.langevin_on, op.lv_z_lo, op.lv_z_hi = 1, 1e-3, 3e-3
    elif name == "vacuum":
        op.collisions_on = 0
    return f, ions, srcs, op, snap, 5


def _run(case, prec, tables, snap, per_call):
    from paper_2609_31258_amd import mucite
    f, ions, srcs, op, _, steps = case
    n = len(snap["x"])
    with mucite.Sim(seed=11, pack_capacity=n + 1000, precision=prec, fp32_tables=tables) as g:
        g.setup(f, ions, srcs if n == N else [], op)
        g.write_packs(snap)
        for k in range(0, steps, per_call):
            g.step(min(per_call, steps - k))
        p, t, e = g.read_packs(), g.read_tallies(), g.read_exits()
    return p, t, e


@pytest.mark.parametrize("name", ["dense", "exits", "species", "sorted", "window", "vacuum"])
@pytest.mark.parametrize("prec,tables", [(0, False), (1, False), (1, True)])
def test_stretch_equals_single_steps(name, prec, tables):
    _say("stretch", name, "fp32" if prec else "fp64", "fp32 tables" if tables else "")
    case = _scenario(name)
    snap = case[4]
    ref, tref, eref = _run(case, prec, tables, snap, 1)
    assert len(np.unique(ref["status"])) == (5 if name == "exits" else 1)
    p, t, e = _run(case, prec, tables, snap, 1000)
    for k in STATE + ("id", "w", "q", "tag"):
        assert np.array_equal(p[k], ref[k]), k
    for k in INTS:
        assert np.array_equal(t[k], tref[k]), k
    assert np.array_equal(e, eref)
    row = {int(i): k for k, i in enumerate(ref["id"])}
    for n in (1, 3, 63, 4097, 8191, 16_385, 32_769, 60_001):
        some = {k: v[:n] for k, v in snap.items()}
        p, t, _ = _run(case, prec, tables, some, 1000)
        at = np.array([row[int(i)] for i in p["id"]])
        for k in STATE:
            assert np.array_equal(p[k], ref[k][at]), (n, k)
        assert t["pack_steps"] <= n * case[5]
        if name != "exits":
            assert t["pack_steps"] == n * case[5]


@pytest.mark.parametrize("prec", [0, 1])
def test_stretch_stops_where_the_capacity_ends(prec):
    """Emission past the pack capacity fails at its own step, the steps before it taken."""
    from paper_2609_31258_amd import mucite
    _say("stretch capacity, precision", prec)
    f, ions, _, op, _ = synth.config_c1()
    src = synth.Source(kind=1, ion=0, current_a=1e-9, packs_per_step=30, n_total=1 << 30)
    with mucite.Sim(seed=3, pack_capacity=100, precision=prec) as g:
        g.setup(f, ions, [src], op)
        with pytest.raises(mucite.MucateError) as err:
            g.step(20)
        assert err.value.code == mucite.MC_ENOMEM
        assert g.info()["step"] == 3 and g.info()["n_slots"] == 90
        assert g.read_tallies()["pack_steps"] == 30 + 60 + 90


def test_steps_without_packs_cost_next_to_nothing():
    """20,000 steps of 300 sources that do not emit and no packs: 17 ms of host work, half a second where each step
    was planned as the first of 32 (the bar leaves a factor of ten to the first)."""
    import time
    from paper_2609_31258_amd import mucite
    _say("steps without packs")
    f, ions, _, op, _ = synth.config_c1()
    srcs = [synth.Source(kind=2, ion=0, current_a=1e-12, weight=1e9, n_total=10) for _ in range(300)]
    with mucite.Sim(seed=1, pack_capacity=100) as g:
        g.setup(f, ions, srcs, op)
        g.step(10)
        best = min(_timed(g, time.perf_counter) for _ in range(3))
        assert g.info()["step"] == 60_010 and g.info()["n_slots"] == 0
    _say(f"  {best * 1e3:.1f} ms")
    assert best < 0.17


def _timed(g, clock):
    t = clock()
    g.step(20_000)
    g.synchronize()
    return clock() - t

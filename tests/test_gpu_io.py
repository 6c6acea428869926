"""Packs through the staging memory: a write and a read give the same values
back (FP64 form bit for bit, FP32 form as pairs of floats), over populations
that take one piece, several, and remainders of both; optional arrays of a
read may be missing."""
import ctypes as C
import sys

import numpy as np
import pytest

from paper_2609_31258_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [1, 255, 257, 21_504, 21_505, 43_009, 120_001])
def test_packs_there_and_back(prec, n):
    from paper_2609_31258_amd import mucite
    print("staged packs", prec, n, flush=True)
    sys.stdout.flush()
    f, _, _, op, _ = synth.config_c1()
    ions = synth.config_c5_species(4)
    snap = synth.pack_snapshot(n, f, seed=n)
    rng = np.random.default_rng(n)
    snap["tag"] = rng.integers(0, 4, n).astype(np.int32)
    snap["w"] = rng.uniform(0.01, 3.0, n)
    snap["h"] = rng.uniform(0.0, 1.0, n)
    with mucite.Sim(seed=1, pack_capacity=n, precision=prec) as g:
        g.setup(f, ions, [], op)
        g.write_packs(snap)
        p = g.read_packs()
        some = mucite.Packs()
        some.n = n
        x, tag = np.zeros(n), np.zeros(n, np.int32)
        some.x, some.tag = mucite._p(x, C.c_double), mucite._p(tag, C.c_int32)
        assert g.L.mc_read_packs(g._h, C.byref(some)) == mucite.MC_OK
        bad = {**snap, "vy": snap["vy"].copy()}
        for v in (np.inf, -np.inf, np.nan):
            bad["vy"][n // 2] = v
            with pytest.raises(mucite.MucateError):
                g.write_packs(bad)
    assert np.array_equal(x, p["x"]) and np.array_equal(tag, snap["tag"])

    def pair(v):
        hi = v.astype(np.float32)
        return hi.astype(np.float64) + (v - hi.astype(np.float64)).astype(np.float32).astype(np.float64)

    for k in ("x", "y", "z", "e_int"):
        assert np.array_equal(p[k], pair(snap[k]) if prec else snap[k]), k
    for k in ("vx", "vy", "vz", "h"):
        assert np.array_equal(p[k], snap[k].astype(np.float32).astype(np.float64) if prec else snap[k]), k
    for k in ("w", "id", "tag"):
        assert np.array_equal(p[k], snap[k]), k
    z = np.array([i.charge_z for i in ions])[snap["tag"]]
    assert np.array_equal(p["q"], np.rint(np.ldexp(z * snap["w"], 32)).astype(np.int64))
    assert not p["status"].any()

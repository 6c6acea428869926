"""The Poisson solve at the edges of its kernels against the oracle: row counts
on both sides of each rows-per-lane class of the tridiagonal scans (2, 4, 8, 16
rows per lane, Thomas sweeps beyond 1024 rows) and of the cyclic
reduction (256 and 512 rows, blocks not full of modes), and row lengths on both sides
of each FFT length.  Bars: FP64 Phi within 1e-10 of max|Phi|, E within 1e-8 of
max|E|; FP32 form (rounding 6e-8 per operation, about 13 butterfly levels in
each of four FFTs) Phi within 5e-6 and E within 1e-4."""
import sys

import numpy as np
import pytest

from paper_2609_31258_amd import synth
from parity_util import make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,nr,nz", [
    (0, 3, 5), (0, 4, 34), (0, 129, 34), (0, 130, 34), (0, 257, 34), (0, 258, 34), (0, 513, 34), (0, 514, 34),
    (0, 1025, 34), (0, 1026, 34), (1, 129, 34), (1, 257, 35), (1, 258, 34), (1, 513, 35), (1, 514, 34), (1, 1025, 34),
    (0, 9, 130), (0, 9, 131), (0, 9, 258), (0, 9, 259), (0, 9, 514), (0, 9, 515), (0, 9, 1026), (0, 9, 1027),
    (0, 9, 2050), (0, 270, 1500), (1, 9, 258), (1, 9, 259), (1, 9, 515), (1, 9, 1027), (1, 9, 2050), (1, 9, 2051)])
def test_poisson_kernel_edges(precision, nr, nz):
    print("poisson edges", precision, nr, nz, flush=True)
    sys.stdout.flush()
    f = synth.uniform_fields(nr, nz, 5e-5)
    op = synth.Operating(dt=1e-9, z_det=f.grid.L, r_det=f.grid.R, sc_on=1)
    snap = synth.pack_snapshot(2000, f, seed=nr + nz, z_lo=0.1 * f.grid.L, z_hi=0.7 * f.grid.L, r_hi=0.6 * f.grid.R)
    for k in ("x", "y", "z"):  # positions that a pair of floats holds exactly
        snap[k] = snap[k].astype(np.float32).astype(np.float64)
    g, o = make_pair(f, [synth.Ion(500.0, 1, 2e-18, 150)], [], op, cap=2000, precision=precision)
    g.write_packs(snap)
    o.write_packs(snap)
    for s in (g, o):
        s.pic_update()
    assert np.array_equal(g.read_charge(), o.read_charge())
    (pa, ra, za), (pb, rb, zb) = g.read_sc(), o.read_sc()
    g.close()
    o.close()
    ep = np.abs(pa - pb).max() / np.abs(pb).max()
    ee = max(np.abs(ra - rb).max(), np.abs(za - zb).max()) / max(np.abs(rb).max(), np.abs(zb).max())
    print(f"  phi {ep:.2e} E {ee:.2e}", flush=True)
    assert ep <= (5e-6 if precision else 1e-10) and ee <= (1e-4 if precision else 1e-8)


@pytest.mark.parametrize("nr,nz,precision", [(3, 1000, 0), (7, 1000, 0), (33, 129, 0), (258, 300, 0), (1026, 64, 0),
                                             (3, 1000, 1), (258, 300, 1)])
def test_device_memory_of_a_context(nr, nz, precision):
    """A context takes no more than its arrays: per node the three static fields and that of the charges (64 bytes),
    potential and charge grids (24), mask and hit bytes, one table record each of field and gas, the modes and two
    coefficients a mode and row for their solve, and the loss map; 128 KiB hold all that does not grow with the grid
    or is that of a row."""
    from paper_2609_31258_amd import mucite
    f = synth.uniform_fields(nr, nz, 5e-5)
    op = synth.Operating(dt=1e-9, z_det=f.grid.L, r_det=f.grid.R, sc_on=1, sc_every=1)
    nn, record, real = nr * nz, (32, 8)[precision], (8, 4)[precision]
    with mucite.Sim(seed=1, pack_capacity=256, precision=precision) as s:
        s.setup(f, [synth.config_c1(10)[1][0]], [], op)
        s.step(1)
        used = s.info()["device_bytes"]
    transform = 2 * real * (5 * nz + 2 * 4 * nz)  # chirp and FFT tables of at most 8 nz points
    print("device memory", nr, nz, precision, used, flush=True)
    assert used <= nn * (64 + 24 + 2 + 2 * record + real + 16 + 8) + transform + 16 * nz + 131_072

"""The deposit's block table where it can go wrong: every cell of a tiny grid
(all corners shared), tables that fill up and overflow into the grid, block
and wavefront remainders.  Both stand-alone entry points, bit for bit against
the oracle's deposit (integer work: the bar is equality)."""
import sys

import numpy as np
import pytest

from test_zz_no_alloc import _case, _gpu_grids, _oracle_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nz,n", [(3, 3, 8), (3, 3, 5000), (4, 5, 1000), (40, 60, 1024), (40, 60, 3000),
                                     (55, 60, 20_001), (130, 300, 1025), (20, 30, 262_145)])
def test_deposit_table(nr, nz, n):
    print("deposit table", nr, nz, n, flush=True)
    sys.stdout.flush()
    f, snap, status, q, charge = _case(nr, nz, n, 40 + nr)
    qa, qb = _gpu_grids(f, snap, status, q)
    want = _oracle_grid(f, snap, status, charge)
    assert np.array_equal(qa, want)
    assert np.array_equal(qb, want)


def test_charge_grid_after_a_refused_mask_update():
    """A space-charge update refused for its mask leaves no charge behind for the next one."""
    from paper_2609_31258_amd import mucite, synth
    f = synth.ring_fields(64, 128)
    f.mask[1:-1, 1:60] = 1  # more interior mask nodes than the correction holds
    snap = synth.pack_snapshot(3000, f, seed=3)
    op = synth.Operating(dt=1e-9, z_det=f.grid.L, r_det=f.grid.R, sc_on=1, sc_mask=1)
    with mucite.Sim(seed=1, pack_capacity=3000) as g:
        g.setup(f, [synth.Ion(500.0, 1, 2e-18, 150)], [], op)
        g.write_packs(snap)
        with pytest.raises(mucite.MucateError) as err:
            g.pic_update()
        assert err.value.code == mucite.MC_EINVAL
        first = g.read_charge()
        op.sc_mask = 0
        g.set_operating(op)
        for _ in range(3):
            g.pic_update()
            assert np.array_equal(g.read_charge(), first)

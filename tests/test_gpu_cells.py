"""Trilinear media: the cells kept in LDS by the integrator against the oracle.
Beams that cross many cells in a launch, wrap around the period, start far
outside the box, share a workgroup with dead beams, or are its ragged tail;
the smallest node grids; c_S from a ratio or a field of its own; samples in
between (the records are written while the next cell is on its way)."""
import numpy as np
import pytest

import oracle as om
from test_gpu_parity import RTOL, compare_states, fga, oracle_to_dict, rel_l2
from test_gpu_smooth_grid import fields, random_beams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(3, 4, 5), (17, 9, 12), (40, 33, 36)])
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("nb, stride", [(1, 1), (63, 2), (65, 3), (200, 1)])
def test_trilinear_cells(n, two, nb, stride):
    m = fga()
    ms, cp, cs = fields(n, 21)
    kw = dict(cs_nodes=cs) if two else dict(cs_ratio=0.58)
    mo, mg = om.grid(cp, ms, **kw), m.Medium.grid(cp, ms, **kw)
    ob = random_beams(nb, -1.3, 2.2, 40 + nb)
    ob["Q"][0] = (900.25, -700.5, 3.0)
    dead = np.arange(nb) % 7 == 3
    ob["alive"][dead] = 0
    bs = m.BeamSet(nb + 5)
    bs.load(oracle_to_dict(ob))
    rec = np.random.default_rng(2).random((5, 3)) * 2.0 - 0.5
    eps = 1.0 / 16
    seis, _ = m.fga_evolve(mg, bs, 8e-3, 12, receivers=rec, eps=eps, stride=stride, chunk=7)
    ob = ob[~dead]
    ref = np.zeros((5, 12 // stride, 3), dtype=np.complex128)
    for s in range(12):
        om.evolve(mo, ob, 8e-3, 1)
        if (s + 1) % stride == 0:
            ref[:, (s + 1) // stride - 1], _ = om.sum_points(ob, rec, eps, 25.0)
    d = bs.export()
    live = (d["flags"] & m.FGA_FLAG_ALIVE) != 0
    compare_states({k: v[live] for k, v in d.items()}, ob)
    assert rel_l2(m.to_complex(seis), ref) <= RTOL or np.abs(ref).max() == 0.0

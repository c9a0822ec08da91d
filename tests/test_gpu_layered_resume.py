"""Layered media: a beam's state does not depend on the chunk, bit for bit, over
flat and spherical layers with and without free surfaces, gradients and the
crosswell model, also where children fall into a later receiver batch.  The
seismograms differ by the order of their sums."""
import numpy as np
import pytest

import fga_inputs as fi
from test_gpu_parity import layered_case, oracle_to_dict

pytestmark = pytest.mark.gpu

STEPS = 40


def start(name):
    import paper_1810_06760_amd as m
    if name != "crosswell":
        _, ob, _, med = layered_case(name)
        b = m.BeamSet(8 * len(ob))
        b.load(oracle_to_dict(ob))
        lo, hi = ob["Q"].min(axis=0), ob["Q"].max(axis=0)
        return med, b, lo + (hi - lo) * np.random.default_rng(3).random((5, 3)), 1.0 / 32, 0.005
    # a shallow source: beams reach the surface, the anomaly layer and the interface below it
    c = fi.crosswell(source=3, eps=1.0 / 64)
    med = m.Medium.layered(0, c["bounds"], c["cp"], c["cs"], c["rho"], surface=c["surface"], anomaly=c["anomaly"])
    src = m.point_source(c["eps"], c["x0"], c["M"], nq=3, ndir=40, nshell=3, ricker=True, merge_s=True)
    first = m.fga_decompose_point_source(med, src).export()
    b = m.BeamSet(12 * len(first["lineage"]))
    b.load(first)
    return med, b, c["receivers"][::4] * np.array([0.2, 1.0, 1.0]), c["eps"], 0.02


def solve(name, chunk, batch, stride, s_vector):
    import paper_1810_06760_amd as m
    med, b, rec, eps, dt = start(name)
    n0 = b.count
    seis, st = m.fga_evolve(med, b, dt, STEPS, receivers=rec, eps=eps, stride=stride, chunk=chunk,
                            batch=batch and max(64, n0 // batch), resort=-1, s_vector=s_vector, cutoff_abs=1e-9)
    n = b.count
    alive = (b.i32[m.FGA_FLAGS, :n] & m.FGA_FLAG_ALIVE).nonzero().ravel()
    alive = alive[b.lineage[:n][alive].argsort()]
    return b.f64[:, alive], b.i32[:, alive], b.lineage[alive], seis, st, n0


# batch: the receiver batch as a fraction of the first beams (0: all beams in one)
@pytest.mark.parametrize("chunk, batch, stride", [(16, 0, 1), (STEPS, 3, 4), (7, 5, 2)])
@pytest.mark.parametrize("name, s_vector", [("flat", False), ("sphere_free", False), ("flat_grad", True),
                                            ("sphere_grad", False), ("flat_anom", True), ("crosswell", False),
                                            ("crosswell", True)])
def test_states_do_not_depend_on_the_chunk(name, s_vector, chunk, batch, stride):
    import torch
    one = solve(name, 1, 0, stride, s_vector)
    got = solve(name, chunk, batch, stride, s_vector)
    assert one[4]["crossings"] > 50 and one[4]["spawned"] > 50
    for k in ("beam_steps", "evals", "crossings", "spawned", "capped", "culled", "quarantined"):
        assert got[4][k] == one[4][k], k
    for a, c in zip(got[:3], one[:3]):
        assert torch.equal(a, c)
    # sums of the same terms in another order
    assert float((got[3] - one[3]).abs().max()) <= 1e-12 * float(one[3].abs().max())
    assert float(one[3].abs().max()) > 0.0

"""Layered media: the steps of a chunk against one step at a time, over chunks,
receiver batches that children fall out of, strides and media."""
import numpy as np
import pytest

from test_gpu_parity import layered_case, oracle_to_dict

pytestmark = pytest.mark.gpu

STEPS = 37


def solve(name, chunk, batch, stride, resort, s_vector, cutoff):
    import paper_1810_06760_amd as m
    w, ob, _, med = layered_case(name)
    b = m.BeamSet(8 * len(ob))
    b.load(oracle_to_dict(ob))
    lo, hi = ob["Q"].min(axis=0), ob["Q"].max(axis=0)
    rec = lo + (hi - lo) * np.random.default_rng(3).random((5, 3))
    seis, st = m.fga_evolve(med, b, 0.005, STEPS, receivers=rec, eps=1.0 / 32, stride=stride, chunk=chunk, batch=batch,
                            resort=resort, s_vector=s_vector, cutoff_abs=cutoff)
    n = b.count
    flags = b.i32[m.FGA_FLAGS, :n]
    assert bool(((flags & ~3) == 0).all())  # alive or quarantined and nothing else
    idx = (flags & m.FGA_FLAG_ALIVE).nonzero().ravel()
    idx = idx[b.lineage[:n][idx].argsort()]
    return b.f64[:, idx].cpu(), b.i32[:, idx].cpu(), b.lineage[idx].cpu(), seis.cpu(), st


@pytest.mark.parametrize("name, s_vector", [("flat", False), ("sphere", False), ("flat_grad", True)])
@pytest.mark.parametrize("chunk, batch, stride, resort", [(16, 0, 1, -1), (5, 64, 2, -1), (0, 100, 3, 7),
                                                          (STEPS, 0, 4, 0)])
def test_chunks_match_single_steps(name, s_vector, chunk, batch, stride, resort):
    one = solve(name, 1, 0, stride, -1, s_vector, 1e-7)
    got = solve(name, chunk, batch, stride, resort, s_vector, 1e-7)
    assert one[4]["crossings"] > 0
    for k in ("beam_steps", "evals", "crossings", "spawned", "capped", "culled", "quarantined"):
        assert got[4][k] == one[4][k], k
    for a, c in zip(got[1:3], one[1:3]):
        assert a.equal(c)
    # the same arithmetic a beam up to the order of sums: 37 steps of a few hundred roundings
    scale = one[0].abs().amax(dim=1, keepdim=True) + 1e-300
    assert float(((got[0] - one[0]).abs() / scale).max()) < 1e-10
    assert float((got[3] - one[3]).abs().max()) < 1e-10 * float(one[3].abs().max())

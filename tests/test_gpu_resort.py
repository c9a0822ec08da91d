"""Spatial re-ordering of the beam set: the planes travel with their beams
whatever scratch the call has (no receivers: a few planes; receivers sampled
every step of a one-step launch: some twenty; the default: all at once)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def random_beams(m, n, seed):
    import torch
    g = np.random.default_rng(seed)
    b = m.BeamSet(n + 3)
    f = g.standard_normal((m.FGA_NF64, n))
    f[m.FGA_Q:m.FGA_Q + 3] = g.random((3, n))
    f[m.FGA_P:m.FGA_P + 3] += 2.0
    f[m.FGA_ZQ_RE:m.FGA_ZQ_RE + 9] = np.eye(3).reshape(9, 1) + 0.1 * g.standard_normal((9, n))
    f[m.FGA_ZP_IM:m.FGA_ZP_IM + 9] = -np.eye(3).reshape(9, 1)
    f[m.FGA_E:m.FGA_E + 3] = np.array([[0.0], [0.0], [1.0]])
    i = np.zeros((m.FGA_NI32, n), dtype=np.int32)
    i[m.FGA_BRANCH] = g.integers(0, 2, n)
    i[m.FGA_SIGMA] = 1
    i[m.FGA_GEN] = g.integers(0, 4, n)
    i[m.FGA_FLAGS] = np.where(g.random(n) < 0.8, m.FGA_FLAG_ALIVE, 0)
    i[m.FGA_FLAGS, 0] = m.FGA_FLAG_ALIVE
    b.f64[:, :n] = torch.from_numpy(f).cuda()
    b.i32[:, :n] = torch.from_numpy(i).cuda()
    b.lineage[:n] = torch.from_numpy(g.permutation(n)).cuda()
    b.c.count = n
    return b


def planes_by_lineage(m, b):
    n = b.count
    live = (b.i32[m.FGA_FLAGS, :n] & m.FGA_FLAG_ALIVE) != 0
    idx = live.nonzero().ravel()
    idx = idx[b.lineage[:n][idx].argsort()]
    return b.f64[:, idx], b.i32[:, idx], b.lineage[idx]


@pytest.mark.parametrize("n", [1, 20, 255, 257, 5000])
@pytest.mark.parametrize("receivers, chunk", [(0, 0), (3, 1), (3, 0)])
def test_reordering_keeps_beams_whole(n, receivers, chunk):
    """Two sorts (one per step) against the same steps without any, bitwise per lineage; dead beams leave."""
    import torch
    import paper_1810_06760_amd as m
    med = m.Medium.homogeneous(1.7, 1.0)
    rec = np.random.default_rng(1).random((receivers, 3)) if receivers else None
    got = {}
    for resort in (1, -1):
        b = random_beams(m, n, 7 + n)
        m.fga_evolve(med, b, 1e-3, 2, receivers=rec, eps=1.0 / 16, chunk=chunk or 1 if resort > 0 else chunk,
                     resort=resort)
        got[resort] = planes_by_lineage(m, b)
        if resort > 0:
            assert b.count == got[1][2].numel()
    for a, c in zip(got[1], got[-1]):
        assert torch.equal(a, c)

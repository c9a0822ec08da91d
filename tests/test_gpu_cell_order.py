"""A beam's steps in a trilinear medium do not depend on the beams beside it: the
same set in order of place (neighbours share cells and the cache lines they are
fetched from) and in the order given, bitwise."""
import pytest

from test_gpu_resort import planes_by_lineage, random_beams
from test_gpu_smooth_grid import fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, nodes, dt", [(400000, 16, 4e-3), (1000000, 64, 2e-3), (200000, 8, 2e-2)])
@pytest.mark.parametrize("s_vector", [False, True])
def test_order_does_not_matter(n, nodes, dt, s_vector):
    import torch
    import paper_1810_06760_amd as m
    ms, cp, _ = fields((nodes, nodes, nodes), 21)
    med = m.Medium.grid(cp, ms, cs_ratio=0.6)
    got = {}
    for resort in (1, -1):
        b = random_beams(m, n, 11)
        m.fga_evolve(med, b, dt, 32, chunk=32, resort=resort, s_vector=s_vector)
        got[resort] = planes_by_lineage(m, b)
    for a, d in zip(got[1], got[-1]):
        assert torch.equal(a, d)

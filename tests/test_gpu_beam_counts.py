"""fga_beams_info around the edges of its grid, against the planes themselves."""
import pytest

from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 257, 65535, 65537, 200001])
def test_counts(n):
    import torch
    import paper_1810_06760_amd as m
    b = random_beams(m, n, n)
    quar = torch.arange(n, device="cuda") % 7 == 3
    flags = b.i32[m.FGA_FLAGS, :n]
    flags[quar] = m.FGA_FLAG_QUARANTINED
    alive = (flags & m.FGA_FLAG_ALIVE) != 0
    br, gen = b.i32[m.FGA_BRANCH, :n], b.i32[m.FGA_GEN, :n]
    got = b.info()
    assert got["alive"] == int(alive.sum())
    assert got["quarantined"] == int(quar.sum())
    assert got["by_branch"] == [int((alive & (br == k)).sum()) for k in range(3)]
    assert got["children"] == int((alive & (gen > 0)).sum())

"""The points' own ordering before a sum: any order of the same points gives the
same sums, bitwise; a point that is not finite is refused by its index."""
import numpy as np
import pytest

from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu


# around a workgroup of points and the most that are ordered on the device; repeated and collinear points
@pytest.mark.parametrize("points", [1, 2, 255, 256, 257, 999, 1024, 1025])
def test_order_of_points(points):
    import torch
    import paper_1810_06760_amd as m
    b = random_beams(m, 3000, 9)
    g = np.random.default_rng(points)
    x = g.random((points, 3))
    x[points // 2:] = x[: points - points // 2]      # every second point twice
    x[: points // 4, 2] = 0.25                       # a plane of points
    want, count = m.fga_reconstruct_points(b, 1.0 / 64, 25.0, x)
    p = g.permutation(points)
    got, count2 = m.fga_reconstruct_points(b, 1.0 / 64, 25.0, x[p])
    assert count2 == count
    assert torch.equal(got, want[torch.from_numpy(p).cuda()])
    for k in {0, points // 2, points - 1}:
        y = x.copy()
        y[k, k % 3] = np.nan if k % 2 else np.inf
        with pytest.raises(Exception, match="point %d is not finite" % k):
            m.fga_reconstruct_points(b, 1.0 / 64, 25.0, y)

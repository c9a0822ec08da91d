"""The Gaussian's exponent in FP64 point sums carries no error common to all
terms: single terms against exponentials of 40 digits."""
import math
from decimal import Decimal, getcontext

import numpy as np
import pytest

from test_gpu_points_wide import one_beam

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 300000])   # the one-launch sum without allocation, and the general one
@pytest.mark.parametrize("eps", [1.0 / 128, 1.0 / 300, 0.0073, 0.01])
def test_exponents_are_unbiased(n, eps):
    """A scale rounded to 53 bits shifts every exponent g by the same share, up to 2^-53.  Bound on the mean
    relative error: 2^-57 of the mean g (115).  What is left rounds either way: |x - Q|^2, 2^-53 of g a term,
    2^-59 of it over 4000, and the exponential itself, an ulp a term."""
    import torch
    import paper_1810_06760_amd as m
    getcontext().prec = 40
    tau, points = 230.0, 4000
    rng = np.random.default_rng(11)
    r = np.sqrt(2.0 * eps * 0.98 * tau * rng.random(points))
    a = 2.0 * math.pi * rng.random(points)
    x = np.stack([np.zeros(points), r * np.cos(a), r * np.sin(a)], axis=1)
    g = [(Decimal(float(y)) ** 2 + Decimal(float(z)) ** 2) / (2 * Decimal(eps)) for _, y, z in x]
    exact = [(-v).exp() for v in g]
    b = one_beam(m, n)
    xd = torch.from_numpy(x).cuda()
    out = torch.empty((points, 3, 2), dtype=torch.float64, device="cuda")
    if n == 1:
        m.fga_reconstruct_points_noalloc(b, eps, tau, xd, out)
    else:
        m.fga_reconstruct_points(b, eps, tau, xd, out=out)
    err = [float((Decimal(float(u)) - w) / w) for u, w in zip(out[:, 0, 0].cpu(), exact)]
    assert abs(sum(err)) <= 2.0 ** -57 * float(sum(g))

"""FP64 point sums in windows so wide that magnitudes leave the normal range:
they go on through the subnormal numbers to exactly 0, as exp does."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def one_beam(m, n):
    """n copies of a unit P beam along x, all but the first without weight."""
    import torch
    b = m.BeamSet(n)
    f = np.zeros((m.FGA_NF64, n))
    f[m.FGA_P] = f[m.FGA_A0_RE] = f[m.FGA_E + 2] = 1.0
    f[m.FGA_ZQ_RE:m.FGA_ZQ_RE + 9] = np.eye(3).reshape(9, 1)
    f[m.FGA_ZP_IM:m.FGA_ZP_IM + 9] = -np.eye(3).reshape(9, 1)
    f[m.FGA_W_RE, 0] = 1.0
    i = np.zeros((m.FGA_NI32, n), dtype=np.int32)
    i[m.FGA_SIGMA] = 1
    i[m.FGA_FLAGS] = m.FGA_FLAG_ALIVE
    b.f64.copy_(torch.from_numpy(f))
    b.i32.copy_(torch.from_numpy(i))
    b.c.count = n
    return b


# one beam takes the one-launch sum without allocation; the larger set the general one
@pytest.mark.parametrize("n", [1, 300000])
@pytest.mark.parametrize("tau", [234.0, 300.0, 1000.0, 3000.0])
def test_far_terms_underflow(n, tau):
    """Offsets across P (phase 0) with exponents g through 700, the subnormal range and beyond.  Bound: the
    exponent's few roundings, 2^-50 g, of the value, and two of the smallest subnormal."""
    import torch
    import paper_1810_06760_amd as m
    b = one_beam(m, n)
    eps = 1.0 / 128
    g = np.array([1.0, 230.0, 600.0, 699.0, 701.0, 708.0, 715.0, 730.0, 744.0, 746.0, 800.0, 1500.0, 5900.0])
    g = g[g < 1.99 * tau]
    x = np.zeros((len(g), 3))
    x[:, 1] = x[:, 2] = np.sqrt(eps * g)
    t = x[:, 1] ** 2 + x[:, 2] ** 2
    want = np.array([math.exp(-v / (2.0 * eps)) for v in t])
    assert (np.sqrt(eps * g) <= math.sqrt(2.0 * tau * eps)).all()
    xd = torch.from_numpy(x).cuda()
    out = torch.full((len(g), 3, 2), float("nan"), dtype=torch.float64, device="cuda")
    u, _ = m.fga_reconstruct_points(b, eps, tau, xd)
    v, _ = m.fga_reconstruct_points_noalloc(b, eps, tau, xd, out)
    for s in (u, v):
        s = s.cpu().numpy()
        assert (np.abs(s[:, 0, 0] - want) <= 2.0 ** -50 * g * want + 2.0 * 5e-324).all()
        assert (s[g >= 746.0] == 0.0).all() and (s[:, 1:] == 0.0).all()

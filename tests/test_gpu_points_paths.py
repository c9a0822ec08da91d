"""The receiver-sum kernel's paths against a direct double sum: tiles wholly
inside a point's window, partly inside and out of reach; dead beams and a
ragged last tile; few and many points; windows so wide that the smallest
magnitudes leave the normal range; ranges of one tile and of many."""
import math

import numpy as np
import pytest

from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu


def direct(m, b, x, eps, tau):
    n = b.count
    F = b.f64[:, :n].cpu().numpy()
    I = b.i32[:, :n].cpu().numpy()
    keep = (I[m.FGA_FLAGS] & m.FGA_FLAG_ALIVE) != 0
    F, I = F[:, keep], I[:, keep]
    Q, P, e = F[m.FGA_Q:m.FGA_Q + 3].T, F[m.FGA_P:m.FGA_P + 3].T, F[m.FGA_E:m.FGA_E + 3].T
    a0, a1 = F[m.FGA_A0_RE] + 1j * F[m.FGA_A0_IM], F[m.FGA_A1_RE] + 1j * F[m.FGA_A1_IM]
    w = (F[m.FGA_W_RE] + 1j * F[m.FGA_W_IM]) * np.exp(1j * F[m.FGA_S] / eps)
    ph = P / np.linalg.norm(P, axis=1, keepdims=True)
    sh = np.cross(e, P)
    sh /= np.linalg.norm(sh, axis=1, keepdims=True)
    sv = np.cross(ph, sh)
    A = np.where((I[m.FGA_BRANCH] == 0)[:, None], a0[:, None] * ph, a0[:, None] * sv + a1[:, None] * sh)
    d = x[:, None, :] - Q[None]
    inside = np.abs(d).max(-1) <= math.sqrt(2.0 * tau * eps)
    E = np.exp(-(d * d).sum(-1) / (2.0 * eps) + 1j * (d * P[None]).sum(-1) / eps) * inside
    return E @ (w[:, None] * A), int(inside.sum())


@pytest.mark.parametrize("n, points", [(1, 1), (64, 4), (65, 5), (1000, 9), (4097, 65), (70000, 33)])
@pytest.mark.parametrize("tau, eps", [(25.0, 1.0 / 32), (25.0, 1.0 / 4096), (300.0, 1.0 / 2000)])
def test_point_sum_paths(n, points, tau, eps):
    """Bounds: FP64 rounding of a phase of a few thousand radians over the sum (1e-11 of the magnitudes summed);
    FP32 factors 2^-20 each."""
    import torch
    import paper_1810_06760_amd as m
    b = random_beams(m, n, 100 + n)
    # neighbours in memory are neighbours in space, as after a re-ordering
    q = b.f64[m.FGA_Q:m.FGA_Q + 3, :n]
    order = (q[0] * 8).floor() * 64 + (q[1] * 8).floor() * 8 + (q[2] * 8).floor()
    idx = order.argsort(stable=True)
    b.f64[:, :n] = b.f64[:, :n][:, idx].clone()
    b.i32[:, :n] = b.i32[:, :n][:, idx].clone()
    x = np.random.default_rng(5).random((points, 3))
    want, count = direct(m, b, x, eps, tau)
    F = b.f64[:, :n]
    scale = float((F[m.FGA_W_RE:m.FGA_W_RE + 2].norm(dim=0) * F[m.FGA_A0_RE:m.FGA_A0_RE + 4].norm(dim=0)).norm())
    xd = torch.from_numpy(x).cuda()
    out = torch.empty((points, 3, 2), dtype=torch.float64, device="cuda")
    for prec, tol in ((m.FGA_FP64, 1e-11), (m.FGA_FP32, 2.0 ** -18), (m.FGA_FP32_ACC32, 2.0 ** -18)):
        u, evals = m.fga_reconstruct_points(b, eps, tau, x, precision=prec)
        assert evals == count
        assert np.abs(m.to_complex(u) - want).max() <= tol * scale
        u2, ev2 = m.fga_reconstruct_points_noalloc(b, eps, tau, xd, out, precision=prec, want_evals=True)
        assert ev2 == count
        assert np.abs(m.to_complex(u2) - want).max() <= tol * scale
        u3, none = m.fga_reconstruct_points_noalloc(b, eps, tau, xd, out.clone(), precision=prec, want_evals=False)
        assert none is None and torch.equal(u2, u3)

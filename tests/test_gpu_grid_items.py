"""Work items of the grid sum on small grids (one to a few tiles cut into many
candidate segments) against the direct point sum at every grid point."""
import numpy as np
import pytest

import fga_inputs as fi
from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(16, 16, 16), (5, 17, 33)])
@pytest.mark.parametrize("nb", [1, 63, 65, 1023, 40000])
def test_grid_items_match_point_sums(n, nb):
    """FP64: both sums of the same terms, 1e-11 of the weights' norm; split 16-bit products: 2^-14 of it."""
    import torch
    import paper_1810_06760_amd as m
    b = random_beams(m, nb, 300 + nb)
    mesh = fi.Mesh3(n, tuple(0.3 / k for k in n), tuple(0.9 / k for k in n))
    eps, tau = 1.0 / 48, 20.0
    F = b.f64[:, :nb]
    scale = float((F[m.FGA_W_RE:m.FGA_W_RE + 2].norm(dim=0) * F[m.FGA_A0_RE:m.FGA_A0_RE + 4].norm(dim=0)).norm())
    want, count = m.fga_reconstruct_points(b, eps, tau, mesh.points())
    want = m.to_complex(want).T.reshape(3, n[2], n[1], n[0])
    for prec, tol in ((m.FGA_FP64, 1e-11), (m.FGA_FP16X3, 2.0 ** -14)):
        u, evals = m.fga_reconstruct_grid(b, eps, tau, mesh, precision=prec)
        assert evals == count
        assert np.abs(m.to_complex(u) - want).max() <= tol * scale
        u2, _ = m.fga_reconstruct_grid(b, eps, tau, mesh, precision=prec, out=u.clone(), add=True)
        assert torch.allclose(u2, 2.0 * u, rtol=1e-12, atol=0.0)

"""Grid sums at the tile counts where the length of work items changes, against
the direct sum at the grid points: 27 and 45 tiles (at most 512 items), 48 (eight
a tile in FP64) and 60 (eight a tile in the mixed modes too)."""
import numpy as np
import pytest

import fga_inputs as fi
from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(48, 48, 48), (80, 48, 48), (64, 64, 45), (80, 61, 48)])
@pytest.mark.parametrize("nb", [300, 20000])
def test_items_of_few_and_many_tiles(n, nb):
    """FP64: both sums of the same terms, 1e-11 of the weights' norm; split 16-bit products: 2^-14 of it."""
    import paper_1810_06760_amd as m
    b = random_beams(m, nb, 500 + nb)
    mesh = fi.Mesh3(n, tuple(0.3 / k for k in n), tuple(0.9 / k for k in n))
    eps, tau = 1.0 / 256, 20.0
    F = b.f64[:, :nb]
    scale = float((F[m.FGA_W_RE:m.FGA_W_RE + 2].norm(dim=0) * F[m.FGA_A0_RE:m.FGA_A0_RE + 4].norm(dim=0)).norm())
    want, count = m.fga_reconstruct_points(b, eps, tau, mesh.points())
    want = m.to_complex(want).T.reshape(3, n[2], n[1], n[0])
    for prec, tol in ((m.FGA_FP64, 1e-11), (m.FGA_FP16X3, 2.0 ** -14)):
        u, evals = m.fga_reconstruct_grid(b, eps, tau, mesh, precision=prec)
        assert evals == count
        assert np.abs(m.to_complex(u) - want).max() <= tol * scale

"""Grid sums in workspaces that hold fewer partial tiles than the query counts."""
import pytest

import fga_inputs as fi
from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu

TILE = 3 * 16 ** 3 * 16  # bytes of a partial tile


# 8, 27 and 56 tiles; partial tiles less than the query's: down to nine a tile where it counts 512
@pytest.mark.parametrize("n, fewer", [((32, 32, 32), 1), ((32, 32, 32), 512 - 72), ((48, 48, 48), 512 - 243),
                                      ((112, 64, 32), 8)])
def test_fewer_partial_tiles(n, fewer):
    """The same terms in another order: FP64 1e-11 of the weights' norm, split 16-bit products 2^-14."""
    import torch
    import paper_1810_06760_amd as m
    nb = 20000
    b = random_beams(m, nb, 900)
    mesh = fi.Mesh3(n, tuple(0.3 / k for k in n), tuple(0.9 / k for k in n))
    eps, tau = 1.0 / 128, 20.0
    F = b.f64[:, :nb]
    scale = float((F[m.FGA_W_RE:m.FGA_W_RE + 2].norm(dim=0) * F[m.FGA_A0_RE:m.FGA_A0_RE + 4].norm(dim=0)).norm())
    size = m.workspace_bytes("grid", beams=b, mesh=mesh, eps=eps, tau=tau)
    nn, lo, h = (m.C.c_int * 3)(*n), (m.C.c_double * 3)(*mesh.lo), (m.C.c_double * 3)(*mesh.h)
    for prec, tol in ((m.FGA_FP64, 1e-11), (m.FGA_FP16X3, 2.0 ** -14)):
        want, count = m.fga_reconstruct_grid(b, eps, tau, mesh, precision=prec)
        u = torch.full_like(want, float("nan"))
        ws = torch.empty(size - fewer * TILE, dtype=torch.uint8, device="cuda")
        ev = m.C.c_int64(0)
        m._check(m.lib().fga_reconstruct_grid(m.C.byref(b.c), eps, tau, nn, lo, h, prec, m._ptr(u), m._ptr(ws),
                                              ws.numel(), m._stream(), m.C.byref(ev)))
        assert ev.value == count
        assert float((u - want).abs().max()) <= tol * scale


def test_too_small_is_refused():
    import torch
    import paper_1810_06760_amd as m
    n = (32, 32, 32)
    b = random_beams(m, 20000, 900)
    mesh = fi.Mesh3(n, tuple(0.3 / k for k in n), tuple(0.9 / k for k in n))
    size = m.workspace_bytes("grid", beams=b, mesh=mesh, eps=1.0 / 128, tau=20.0)
    nn, lo, h = (m.C.c_int * 3)(*n), (m.C.c_double * 3)(*mesh.lo), (m.C.c_double * 3)(*mesh.h)
    out = torch.empty((3, 32, 32, 32, 2), dtype=torch.float64, device="cuda")
    ws = torch.empty(size - (512 - 72 + 1) * TILE, dtype=torch.uint8, device="cuda")
    assert m.lib().fga_reconstruct_grid(m.C.byref(b.c), 1.0 / 128, 20.0, nn, lo, h, m.FGA_FP64, m._ptr(out), m._ptr(ws),
                                        ws.numel(), m._stream(), None) == 2

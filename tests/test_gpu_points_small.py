"""The one-launch sum of few beams at few points: repeated and captured calls
leave its counters ready for the next, and agree with the general call."""
import pytest

from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu


# one workgroup; one row; the last sizes that take one launch and the first that do not
@pytest.mark.parametrize("n, points", [(1, 1), (256, 5), (257, 4), (3000, 65), (64 * 4 * 256, 16), (64 * 4 * 256 + 1, 16),
                                       (100, 4096), (100, 4097)])
def test_repeats_and_replays(n, points):
    """The two calls sum the same terms in another order: 1e-12 of the magnitudes summed (FP32 terms: the same
    factors, their 32-bit lane sums 64 terms long, 2^-18)."""
    import torch
    import paper_1810_06760_amd as m
    b = random_beams(m, n, 3 + n)
    x = torch.rand(points, 3, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    F = b.f64[:, :n]
    scale = float((F[m.FGA_W_RE:m.FGA_W_RE + 2].norm(dim=0) * F[m.FGA_A0_RE:m.FGA_A0_RE + 4].norm(dim=0)).norm())
    for prec, tol in ((m.FGA_FP64, 1e-12), (m.FGA_FP32, 1e-12), (m.FGA_FP32_ACC32, 2.0 ** -18)):
        want, count = m.fga_reconstruct_points(b, 1.0 / 32, 25.0, x, precision=prec)
        out = torch.full((points, 3, 2), float("nan"), dtype=torch.float64, device="cuda")
        _, ev = m.fga_reconstruct_points_noalloc(b, 1.0 / 32, 25.0, x, out, precision=prec)
        assert ev == count
        assert float((out - want).abs().max()) <= tol * scale
        first = out.clone()
        g = torch.cuda.CUDAGraph()
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            m.fga_reconstruct_points_noalloc(b, 1.0 / 32, 25.0, x, out, precision=prec, want_evals=False)
        torch.cuda.current_stream().wait_stream(s)
        with torch.cuda.graph(g):
            m.fga_reconstruct_points_noalloc(b, 1.0 / 32, 25.0, x, out, precision=prec, want_evals=False)
        for _ in range(4):
            out.fill_(float("nan"))
            g.replay()
            assert torch.equal(out, first)
            torch.cuda.synchronize()
            out.fill_(float("nan"))
            m.fga_reconstruct_points_noalloc(b, 1.0 / 32, 25.0, x, out, precision=prec, want_evals=False)
            assert torch.equal(out, first)

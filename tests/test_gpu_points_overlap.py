"""The one-launch sum's counters after calls that overlapped on the device.
Such calls may spoil each other's results; none spoils a later call's."""
import pytest

from test_gpu_resort import random_beams

pytestmark = pytest.mark.gpu


def test_later_calls_survive_overlapping_ones():
    """Replays of one graph and eager calls of other sizes on four streams at once; then each size by itself,
    bit for bit as before."""
    import torch
    import paper_1810_06760_amd as m
    gen = torch.Generator("cuda").manual_seed(5)
    cases = []
    for n, points in ((300, 4), (3000, 65), (20000, 40), (65536, 16)):   # 2, 12, 79 and 256 rows
        b = random_beams(m, n, n)
        x = torch.rand(points, 3, dtype=torch.float64, device="cuda", generator=gen)
        out = torch.empty((points, 3, 2), dtype=torch.float64, device="cuda")
        cases.append((b, x, out))

    def call(k):
        b, x, out = cases[k]
        m.fga_reconstruct_points_noalloc(b, 1.0 / 32, 25.0, x, out, want_evals=False)

    first = []
    for k in range(4):
        call(k)
        first.append(cases[k][2].clone())
    graphs = []
    for k in range(4):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call(k)
        graphs.append(g)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    for turn in range(64):
        for j, s in enumerate(streams):
            with torch.cuda.stream(s):
                if (turn + j) % 3:
                    graphs[(turn + j // 2) % 4].replay()
                else:
                    call((turn + j) % 4)
    torch.cuda.synchronize()
    for k in range(4):
        for replay in (False, True, False):
            cases[k][2].fill_(float("nan"))
            graphs[k].replay() if replay else call(k)
            assert torch.equal(cases[k][2], first[k])
            torch.cuda.synchronize()

"""The workspace of a point sum serves fewer beams and fewer points: a program
sizes it once and sums a culled or compacted set later."""
import pytest


def beams(m, count):
    b = m.Beams()
    b.capacity, b.count, b.f64, b.i32, b.lineage = count, count, 256, 256, 256
    return b


def query(m, count, n):
    return m.lib().fga_reconstruct_points_workspace_bytes(m.C.byref(beams(m, count)), n)


def test_query_grows_with_beams_and_points():
    import paper_1810_06760_amd as m
    for n in (1, 8, 9, 65, 512, 2000, 20000):
        last = 0
        for count in list(range(1, 20000, 7)) + [2 ** k + d for k in range(15, 24) for d in (-1, 0, 1, 64)]:
            size = query(m, count, n)
            assert size >= last, (count, n)
            last = size
    for count in (1, 700, 14561, 100000, 5000000):
        last = 0
        for n in list(range(1, 300)) + list(range(300, 40000, 83)):
            size = query(m, count, n)
            assert size >= last, (count, n)
            last = size


@pytest.mark.gpu
@pytest.mark.parametrize("size_for, sum_of", [((526, 2000), (519, 2000)), ((2052, 512), (2045, 512)),
                                              ((14568, 65), (14561, 65)), ((100000, 9), (100000, 8)),
                                              ((3000, 17), (2999, 16))])
def test_a_workspace_serves_less(size_for, sum_of):
    """The sum in the larger set's workspace is the sum in its own, bit for bit."""
    import torch
    import paper_1810_06760_amd as m
    from test_gpu_resort import random_beams
    n, points = sum_of
    b = random_beams(m, n, n)
    x = torch.rand(points, 3, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    want, _ = m.fga_reconstruct_points(b, 1.0 / 32, 25.0, x)
    size = query(m, *size_for)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(want)
    status = m.lib().fga_reconstruct_points(m.C.byref(b.c), 1.0 / 32, 25.0, points, m._ptr(x), m.FGA_FP64, m._ptr(out),
                                            m._ptr(ws), size, m._stream(), None)
    assert status == 0, m.lib().fga_last_error()
    assert torch.equal(out, want)

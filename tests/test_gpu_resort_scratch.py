"""Re-ordering with any room for the planes: workspaces between the query's
size and the least one give the same beams, bit for bit; and what a request of
the server holds counts the least."""
import numpy as np
import pytest

from test_gpu_resort import planes_by_lineage, random_beams

pytestmark = pytest.mark.gpu

PLANES = 58  # 52 double planes, 5 int32 planes and the lineage, a slot of 8 bytes a beam each


# sets whose query has room for all planes (up to 2^18 slots), and one beyond
@pytest.mark.parametrize("n", [61, 257, 5000, 300001])
@pytest.mark.parametrize("receivers, stride, batch", [(0, 1, 0), (3, 1, 0), (3, 2, 64), (2, 40, 0)])
@pytest.mark.parametrize("room", [0.0, 0.04, 0.31, 0.8])
def test_any_scratch_keeps_beams_whole(monkeypatch, n, receivers, stride, batch, room):
    import torch
    import paper_1810_06760_amd as m
    med = m.Medium.homogeneous(1.7, 1.0)
    rec = np.random.default_rng(1).random((receivers, 3)) if receivers else None
    slots = (n + 3 + 31) // 32 * 32
    got = []
    for resort in (1, -1):
        b = random_beams(m, n, 7 + n)
        if resort > 0:
            def cut(nbytes, ws=None):
                less = int((1.0 - room) * PLANES * 8 * slots) // 256 * 256 if n < 1 << 18 else 0
                return torch.empty(int(nbytes) - less, dtype=torch.uint8, device="cuda")
            monkeypatch.setattr(m, "_workspace", cut)
        _, st = m.fga_evolve(med, b, 1e-3, 2, receivers=rec, eps=1.0 / 16, stride=stride, batch=batch, chunk=1,
                             resort=resort)
        monkeypatch.undo()
        got.append(planes_by_lineage(m, b) + (st["evals"],))
    assert got[0][3] == got[1][3]
    for a, c in zip(got[0][:3], got[1][:3]):
        assert torch.equal(a, c)


@pytest.mark.parametrize("receivers, stride", [(0, 1), (16, 32)])
def test_request_footprint_counts_the_least(receivers, stride):
    """About 24 bytes a beam for the keys and their sort, 8 for crossings, up to 32 for the sorts' own buffers and,
    with receivers, two samples' records (96 bytes) and boxes: not a copy of the planes (464 bytes)."""
    import torch  # noqa: F401
    import paper_1810_06760_amd as m
    src = m.point_source(1.0 / 32, [0.5] * 3, [1.0, 1.0, 1.0, 0.0, 0.0, 0.0], nq=5, ndir=64, nshell=3, merge_s=True)
    cand = int(m.lib().fga_point_source_candidates(m.C.byref(src)))
    rq = m.make_request(m.Medium.homogeneous(1.7, 1.0), None, None, np.zeros((receivers, 3)), 25.0, 2e-3, 64,
                        stride=stride, source=src)
    beams = cand * (m.FGA_NF64 * 8 + m.FGA_NI32 * 4 + 8)
    assert m.Server.footprint(rq[0]) <= beams + cand * (64 + (2 * 97 if receivers else 0)) + (1 << 17)

"""Performance cases of the FGA library: the calls a user's program makes.

Each case is one call, or one whole solve, through the package's public entry
points, at sizes of the repository's own workloads or below and above them:

  points     the Gaussian sum at scattered points (a few receivers; a slice)
  grid       the Gaussian sum on a uniform grid (FP64 and the mixed variants)
  homog      a homogeneous-medium solve: decompose, evolve, grid
  decompose  the FBI decomposition of two-way data on a gridded medium
  source     a point-source solve in a gridded medium with receivers
  window     the smooth-medium packet: decompose and evolve with receivers
  layered    a point-source solve in the layered spherical Earth
  crosswell  a point-source solve in the crosswell model (anomaly, free surface)
  serve      a batch of forward solves through the request server

Results computed with single-precision factors (the mixed modes) are kept in
single precision, as a program that asks for them stores them; everything else
is FP64.  Beams of a solve are returned in lineage order, the order in which
results are matched.
"""
import math
from types import SimpleNamespace

import torch

import paper_1810_06760_amd as fga

SQRT3 = math.sqrt(3.0)
PRECISION = {"fp64": fga.FGA_FP64, "fp32": fga.FGA_FP32, "fp32_acc32": fga.FGA_FP32_ACC32,
             "bf16x3": fga.FGA_BF16X3, "fp16x3": fga.FGA_FP16X3, "fp16x2": fga.FGA_FP16X2}


def listed():
    return [
        # the smallest call: a handful of receivers and a thinned beam set, no allocation (a serving loop)
        dict(name="points-few", kind="points", beams=3000, points=65, log2ieps=5, tau=25.0, precision="fp64",
             noalloc=True),
        # a vertical slice of scattered points of one snapshot, mixed-precision terms
        dict(name="points-slice", kind="points", beams=400000, points=2000, log2ieps=7, tau=25.0,
             precision="fp32_acc32", noalloc=False),
        # the homogeneous packet at its full size: 98,304 beams, 100 steps, 32^3 grid
        dict(name="homog-packet", kind="homog", nq=8, np=4, ny=64, steps=100, nout=32, log2ieps=5, merge=False),
        # Step 1 alone, displacement and velocity given (two-way), odd quadrature mesh
        dict(name="decompose-two-way", kind="decompose", nq=16, np=7, ny=101, nmed=64, log2ieps=7, smooth=False,
             merge=False),
        # the smallest forward solve of the tomography sweep: eps = 1/64, every step sampled at 512 receivers
        dict(name="source-eps64", kind="source", log2ieps=6, nq=8, ndir=16, nshell=2, nmed=128, smooth=False,
             s_vector=False, two=False, steps=160, stride=1, receivers=512, precision="fp64", merge=True),
        # a mid-size forward solve in the C2 medium, frame-free S amplitudes, mixed receiver sums, every other step
        dict(name="source-cubic-eps128", kind="source", log2ieps=7, nq=8, ndir=65, nshell=4, nmed=96, smooth=True,
             s_vector=True, two=False, steps=32, stride=2, receivers=385, precision="fp32_acc32", merge=True),
        # the benchmark's configuration: 33 M beams in the 128^3 medium, 256 receivers sampled every step
        dict(name="window-eps128", kind="window", nq=32, np=8, ny=128, nmed=128, log2ieps=7, steps=32,
             receivers=256),
        # the layered spherical Earth, a sixteenth of its directions: interface children, 512 stations
        dict(name="layered-earth", kind="layered", log2ieps=8, nq=8, ndir=100, nshell=4, steps=48, receivers=512),
        # the crosswell model: curved rays in the anomaly layer, a free surface, the 32 receivers of a well
        dict(name="crosswell", kind="crosswell", log2ieps=7, nq=6, ndir=160, nshell=4, steps=40, receivers=32),
        # a snapshot on the 128^3 grid in FP64 (matrix cores)
        dict(name="grid-128-fp64", kind="grid", beams=300000, nx=128, ny=128, nz=128, log2ieps=7, tau=25.0,
             precision="fp64"),
        # a 256^3 snapshot at eps = 1/512 in split 16-bit products
        dict(name="grid-256-fp16x3", kind="grid", beams=1000000, nx=256, ny=256, nz=256, log2ieps=9, tau=16.0,
             precision="fp16x3"),
        # six requests of the small tomography sweep through the server, four at a time
        dict(name="serve-six", kind="serve", requests=6, steps=100, slots=4, precision="fp64"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["points", "grid", "homog", "decompose", "source", "window", "layered", "crosswell", "serve"])
    if kind == "points":
        noalloc = rng.random() < 0.3
        return dict(kind=kind, beams=_log(rng, 500, 50000 if noalloc else 1000000),
                    points=_log(rng, 1, 500 if noalloc else 4000), log2ieps=rng.randint(5, 9),
                    tau=rng.choice([16.0, 25.0]), precision=rng.choice(["fp64", "fp32", "fp32_acc32"]),
                    noalloc=noalloc)
    if kind == "grid":
        eps = rng.randint(5, 9)
        n = [_log(rng, 20, 256) for _ in range(3)]
        most = 1.2e12 / (n[0] * n[1] * n[2])   # (beam, point) pairs
        return dict(kind=kind, beams=int(min(1000000, max(200, rng.uniform(0.1, 1.0) * most))), nx=n[0], ny=n[1],
                    nz=n[2], log2ieps=eps, tau=rng.choice([16.0, 25.0]),
                    precision=rng.choice(["fp64", "fp64", "fp32", "bf16x3", "fp16x3", "fp16x2"]))
    if kind == "homog":
        return dict(kind=kind, nq=rng.randint(3, 12), np=rng.randint(2, 4), ny=rng.randint(24, 72),
                    steps=_log(rng, 10, 150), nout=rng.randint(12, 40), log2ieps=5, merge=rng.random() < 0.5)
    if kind == "decompose":
        return dict(kind=kind, nq=rng.randint(4, 18), np=rng.randint(3, 8), ny=rng.randint(32, 128),
                    nmed=rng.randint(24, 96), log2ieps=rng.randint(5, 7), smooth=rng.random() < 0.5,
                    merge=rng.random() < 0.5)
    if kind == "source":
        smooth = rng.random() < 0.4
        return dict(kind=kind, log2ieps=rng.randint(5, 8), nq=rng.randint(4, 8), ndir=_log(rng, 12, 300),
                    nshell=rng.randint(1, 4), nmed=rng.randint(32, 128), smooth=smooth,
                    s_vector=rng.random() < 0.4, two=rng.random() < 0.25, steps=_log(rng, 16, 128),
                    stride=rng.choice([1, 1, 2, 5]), receivers=_log(rng, 32, 1024),
                    precision=rng.choice(["fp64", "fp64", "fp32", "fp32_acc32"]), merge=rng.random() < 0.7)
    if kind == "window":
        nq = rng.randint(8, 30)
        return dict(kind=kind, nq=nq, np=rng.randint(4, 8), ny=rng.randint(64, 128), nmed=rng.randint(64, 128),
                    log2ieps=7, steps=rng.randint(8, 34), receivers=rng.choice([0, _log(rng, 64, 512)]))
    if kind == "layered":
        return dict(kind=kind, log2ieps=rng.randint(6, 8), nq=rng.randint(4, 8), ndir=_log(rng, 16, 120),
                    nshell=rng.randint(2, 4), steps=_log(rng, 12, 60), receivers=_log(rng, 64, 600))
    if kind == "crosswell":
        return dict(kind=kind, log2ieps=rng.randint(6, 8), nq=rng.randint(4, 7), ndir=_log(rng, 16, 180),
                    nshell=rng.randint(2, 4), steps=_log(rng, 12, 50), receivers=_log(rng, 8, 64))
    return dict(kind="serve", requests=rng.randint(3, 8), steps=_log(rng, 30, 120), slots=rng.randint(1, 4),
                precision=rng.choice(["fp64", "fp32", "fp32_acc32"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed, purpose):
    g = torch.Generator(device=_device())
    g.manual_seed(1000 * int(seed) + purpose)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, dtype=torch.float64, device=_device(), generator=g)


def _uniform(g, *shape):
    return torch.rand(*shape, dtype=torch.float64, device=_device(), generator=g)


def _mesh(n, lo, h):
    return SimpleNamespace(n=tuple(n), lo=tuple(float(v) for v in lo), h=tuple(float(v) for v in h))


def _cells(n, a, b):
    """Cell-centred points of [a, b], n per axis (n: one number or three)."""
    n = (n,) * 3 if isinstance(n, int) else n
    h = [(b - a) / k for k in n]
    return _mesh(n, [a + 0.5 * v for v in h], h)


def _nodes(n):
    return _mesh((n,) * 3, (0.0,) * 3, (1.0 / n,) * 3)


def _p_mesh(eps, n, width=0.1):
    """n^3 cell-centred p points around (1, 0, 0), +-3 spreads of the packet's transform."""
    half = 3.0 * eps * math.sqrt(1.0 / width ** 2 + 1.0 / eps)
    h = 2.0 * half / n
    return _mesh((n,) * 3, [c - half + 0.5 * h for c in (1.0, 0.0, 0.0)], (h,) * 3)


def _axis(m, d):
    return m.lo[d] + m.h[d] * torch.arange(m.n[d], dtype=torch.float64, device=_device())


def _packet(ymesh, eps, seed, purpose, width=0.1):
    """Gaussian-enveloped plane wave of a random polarisation, complex [3][z][y][x]."""
    d = _normal(_gen(seed, purpose), 3)
    d = d / d.norm()
    x, y, z = _axis(ymesh, 0)[None, None, :], _axis(ymesh, 1)[None, :, None], _axis(ymesh, 2)[:, None, None]
    r2 = (x - 0.5) ** 2 + (y - 0.5) ** 2 + (z - 0.5) ** 2
    s = torch.polar(torch.exp(-r2 / (2.0 * width ** 2)), (x / eps).expand_as(r2).contiguous())
    return d[:, None, None, None].to(torch.complex128) * s[None]


def _field(n, seed, purpose, corr=0.2):
    """c_P nodes of the smooth random medium: sqrt(3) (1 + 0.2 g), g a periodic Gaussian random field of
    correlation length 0.2, standard deviation 1/3, clipped to |g| <= 1."""
    noise = _normal(_gen(seed, purpose), n, n, n)
    k = 2.0 * math.pi * torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=_device())
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2
    f = torch.fft.ifftn(torch.fft.fftn(noise) * torch.exp(-corr ** 2 * k2 / 4.0)).real
    f = f - f.mean()
    f = (f * (1.0 / 3.0 / f.std())).clamp(-1.0, 1.0)
    return (SQRT3 * (1.0 + 0.2 * f)).contiguous()


def _fields(case, seed):
    """c_P nodes, and c_S nodes or None (c_S = c_P/sqrt(3))."""
    cp = _field(case["nmed"], seed, 1)
    return cp, (_field(case["nmed"], seed, 2) / SQRT3 if case.get("two") else None)


def _cull(case):
    """The packet's cull where only the field is wanted; every candidate where the beams are."""
    return 1e-10 * (2.0 * math.pi * 0.1 ** 2) ** 1.5 if case["kind"] == "window" and case["receivers"] else 0.0


def _moment(seed, purpose):
    a = _normal(_gen(seed, purpose), 3, 3)
    m = 0.5 * (a + a.T)
    m = (m / m.norm()).tolist()
    return [m[0][0], m[1][1], m[2][2], m[0][1], m[0][2], m[1][2]]


def _beam_planes(case, seed):
    """A snapshot's beams: centres spread like the packet's, P around (1, 0, 0), P and merged-S amplitudes."""
    n, eps = case["beams"], 2.0 ** -case["log2ieps"]
    g = _gen(seed, 5)
    f = torch.zeros((fga.FGA_NF64, n), dtype=torch.float64, device=_device())
    spread = math.sqrt(0.1 ** 2 + eps)
    f[fga.FGA_Q:fga.FGA_Q + 3] = 0.5 + spread * _normal(g, 3, n)
    f[fga.FGA_P:fga.FGA_P + 3] = eps * math.sqrt(100.0 + 1.0 / eps) * _normal(g, 3, n)
    f[fga.FGA_P] += 1.0
    s = torch.arange(n, device=_device()) % 2
    f[fga.FGA_A0_RE:fga.FGA_A0_RE + 4] = _normal(g, 4, n)
    f[fga.FGA_A1_RE:fga.FGA_A1_RE + 2] *= s
    f[fga.FGA_S] = 0.0
    f[fga.FGA_W_RE:fga.FGA_W_RE + 2] = _normal(g, 2, n) * torch.exp(-3.0 * _uniform(g, 1, n))
    f[fga.FGA_E + 2] = 1.0
    i = torch.zeros((fga.FGA_NI32, n), dtype=torch.int32, device=_device())
    i[fga.FGA_BRANCH] = s.to(torch.int32)
    i[fga.FGA_SIGMA] = 1
    i[fga.FGA_FLAGS] = fga.FGA_FLAG_ALIVE
    return f, i


def _grid_mesh(case):
    return _cells((case["nx"], case["ny"], case["nz"]), 0.0, 1.0)


def _receivers(case, seed):
    return _uniform(_gen(seed, 3), case["receivers"], 3)


def _source_spec(case, seed):
    u = _uniform(_gen(seed, 4), 3)
    return dict(eps=2.0 ** -case["log2ieps"], x0=(0.25 + 0.5 * u).tolist(), M=_moment(seed, 6), nq=case["nq"],
                ndir=case["ndir"], nshell=case["nshell"], merge_s=case["merge"])


def _earth(case, seed):
    """The layered spherical Earth: three interfaces, speeds and densities growing inwards, a source at depth."""
    u = _uniform(_gen(seed, 7), 16).tolist()
    bounds = [0.85 + 0.1 * u[0], 0.6 + 0.1 * u[1], 0.35 + 0.1 * u[2]]
    cp, cs, rho = [SQRT3], [1.0], [1.0]
    for k in range(3):
        cp.append(cp[-1] * (1.05 + 0.15 * u[3 + 3 * k]))
        cs.append(cs[-1] * (1.05 + 0.15 * u[4 + 3 * k]))
        rho.append(rho[-1] * (1.05 + 0.15 * u[5 + 3 * k]))
    d = _normal(_gen(seed, 8), 3)
    x0 = (d / d.norm() * (0.6 + 0.3 * u[12])).tolist()
    n = case["receivers"]
    i = torch.arange(n, dtype=torch.float64, device=_device())
    lat = torch.asin(1.0 - (2.0 * i + 1.0) / n)
    lon = torch.remainder(i * math.pi * (3.0 - math.sqrt(5.0)) + 2.0 * math.pi * u[13], 2.0 * math.pi) - math.pi
    return bounds, cp, cs, rho, x0, torch.stack([torch.ones_like(lat), lon, lat], dim=1).contiguous()


class _Server:
    """The server of one program, closed with it."""

    def __init__(self, budget, slots):
        self.server = fga.Server(budget, slots)

    def __del__(self):
        try:
            self.server.close()
        except Exception:
            pass


# (q points per axis, directions, shells) of the small sweep's requests
SWEEP = {5: (5, 64, 3), 6: (6, 120, 4)}


def _requests(case, seed):
    u = _uniform(_gen(seed, 9), case["requests"], 3).tolist()
    out = []
    for k, v in enumerate(u):
        le = 5 + (k % 2)
        nq, ndir, nshell = SWEEP[le]
        out.append(dict(eps=2.0 ** -le, x0=[0.25 + 0.5 * t for t in v], M=_moment(seed, 20 + k), nq=nq, ndir=ndir,
                        nshell=nshell, merge_s=True, receivers=_uniform(_gen(seed, 40 + k), 128 + 554 * k % 897, 3)))
    return out


def _beam_set(n):
    return fga.BeamSet(n)


def _source_set(src, times=1):
    return _beam_set(times * int(fga.lib().fga_point_source_candidates(fga.C.byref(src))))


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if kind == "serve":
        cp = _field(64, seed, 1)
        s["medium"] = fga.Medium.grid(cp, _nodes(64), cs_ratio=1.0 / SQRT3)
        s["requests"] = []
        for r in _requests(case, seed):
            x = r.pop("receivers").cpu().numpy()
            src = fga.point_source(**r)
            s["requests"].append(fga.make_request(s["medium"], None, None, x, 25.0, 2e-3, case["steps"],
                                                  precision=PRECISION[case["precision"]], source=src))
        most = max(fga.Server.footprint(q[0]) for q in s["requests"])
        s["server"] = _Server(most * case["slots"], case["slots"])
        return s
    eps = 2.0 ** -case["log2ieps"]
    s["eps"] = eps
    if kind in ("points", "grid"):
        b = _beam_set(case["beams"])
        f, i = _beam_planes(case, seed)
        b.f64.copy_(f)
        b.i32.copy_(i)
        b.lineage.copy_(torch.arange(case["beams"], device=_device()))
        b.c.count = case["beams"]
        s["beams"] = b
        if kind == "points":
            s["xyz"] = _uniform(_gen(seed, 3), case["points"], 3)
            s["out"] = torch.empty((case["points"], 3, 2), dtype=torch.float64, device="cuda")
        else:
            s["mesh"] = _grid_mesh(case)
            s["out"] = torch.empty((3, case["nz"], case["ny"], case["nx"], 2), dtype=torch.float64, device="cuda")
            s["ws"] = fga._workspace(fga.workspace_bytes("grid", beams=b, mesh=s["mesh"], eps=eps, tau=case["tau"]))
        return s
    if kind in ("homog", "decompose", "window"):
        y = _cells(case["ny"], 0.0, 1.0)
        s["f"] = torch.view_as_real(_packet(y, eps, seed, 10)).reshape(-1).contiguous()
        if kind == "homog":
            s["medium"] = fga.Medium.homogeneous(SQRT3, 1.0)
        else:
            cp, cs = _fields(case, seed)
            s["medium"] = fga.Medium.grid(cp, _nodes(case["nmed"]), cs_ratio=1.0 / SQRT3, cs_nodes=cs,
                                          smooth=case.get("smooth", False))
        if kind == "decompose":
            s["g"] = torch.view_as_real(_packet(y, eps, seed, 11) / eps).reshape(-1).contiguous()
        merge = case.get("merge", True)
        s["mesh"] = fga.make_mesh(eps, _cells(case["nq"], 0.0, 1.0), _p_mesh(eps, case["np"]), y,
                                  one_way=kind != "decompose", cull_abs=_cull(case),
                                  merge_s=merge)
        n = case["nq"] ** 3 * case["np"] ** 3 * (2 if merge else 3) * (2 if kind == "decompose" else 1)
        s["ws"] = fga._workspace(fga.workspace_bytes("decompose", mesh=s["mesh"], with_g=kind == "decompose"))
        s["dt"], nrec, stride = (0.005, 0, 1) if kind == "homog" else (1e-3, case.get("receivers", 0), 1)
        if kind == "homog":
            s["grid"] = _cells(case["nout"], 0.0, 1.0)
        s["beams"] = _beam_set(n)
        s["rec"] = _receivers(case, seed) if nrec else None
        coords = fga.FGA_COORDS_CARTESIAN
    else:
        coords, stride, s["dt"] = fga.FGA_COORDS_CARTESIAN, case.get("stride", 1), 1e-3
        if kind == "source":
            cp, cs = _fields(case, seed)
            s["medium"] = fga.Medium.grid(cp, _nodes(case["nmed"]), cs_ratio=1.0 / SQRT3, cs_nodes=cs,
                                          smooth=case["smooth"])
            s["src"] = fga.point_source(**_source_spec(case, seed))
            s["rec"] = _receivers(case, seed)
            s["beams"] = _source_set(s["src"])
        elif kind == "layered":
            bounds, cp, cs, rho, x0, s["rec"] = _earth(case, seed)
            s["medium"] = fga.Medium.layered(1, bounds, cp, cs, rho)
            s["src"] = fga.point_source(eps, x0, _moment(seed, 6), nq=case["nq"], ndir=case["ndir"],
                                        nshell=case["nshell"], merge_s=True)
            s["beams"], s["dt"], coords = _source_set(s["src"], 6), 7.5e-4, fga.FGA_COORDS_SPHERICAL
        else:
            cp = [2.2, 2.0, 1.8]
            u = _uniform(_gen(seed, 4), 2).tolist()
            s["medium"] = fga.Medium.layered(0, [1.0, 2.0], cp, [c / SQRT3 for c in cp], [1.0] * 3, surface=3.0,
                                             anomaly={1: (0.1, 1.0e4 / 450.0, (0.75, 0.0, 1.5), (1.0, 0.0, 1.0))})
            s["src"] = fga.point_source(eps, [0.0, 0.0, 3.0 - (0.08 + 2.4 * u[0])], [1.0, 1.0, 1.0, 0.0, 0.0, 0.0],
                                        nq=case["nq"], ndir=case["ndir"], nshell=case["nshell"], merge_s=True)
            z = torch.linspace(2.96, 0.48, case["receivers"], dtype=torch.float64, device=_device())
            s["rec"] = torch.stack([torch.full_like(z, 1.5 - 0.8 * u[1]), torch.zeros_like(z), z], dim=1).contiguous()
            s["beams"] = _source_set(s["src"], 6)
    if kind != "decompose":
        s["coords"], s["stride"] = coords, stride
        n = 0 if s["rec"] is None else s["rec"].shape[0]
        s["ews"] = fga._workspace(fga.workspace_bytes(
            "evolve", beams=s["beams"], nsteps=case["steps"], n_receivers=n, eps=eps, stride=stride, coords=coords,
            precision=PRECISION[case.get("precision", "fp64")]))
        if n:
            s["seis"] = torch.empty((n, case["steps"] // stride, 3, 2), dtype=torch.float64, device="cuda")
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _kept(out, precision):
    return out if precision == "fp64" else out.to(torch.float32)


def _parts(f):
    """The planes as rays and Jacobians, amplitudes and action, weights, frame axes."""
    return {"rays": f[:fga.FGA_A0_RE], "amplitudes": f[fga.FGA_A0_RE:fga.FGA_W_RE],
            "weights": f[fga.FGA_W_RE:fga.FGA_E], "axes": f[fga.FGA_E:]}


def _by_lineage(beams):
    n = beams.count
    return _parts(beams.f64[:, :n].index_select(1, torch.argsort(beams.lineage[:n])))


def run(s):
    case, kind = s["case"], s["kind"]
    if kind == "serve":
        srv = s["server"].server
        for req, _, keep in s["requests"]:
            srv.submit(req, keep)
        left = len(s["requests"])
        while left:
            done = srv.poll(max_n=left, wait_ms=1000)
            for d in done:
                if d["status"] != 0:
                    raise RuntimeError("request %d ended with status %d" % (d["id"], d["status"]))
            left -= len(done)
        seis = [q[1] for q in s["requests"]]
        return seis if case["precision"] == "fp64" else [a.astype("complex64") for a in seis]
    if kind == "points":
        p = PRECISION[case["precision"]]
        if case["noalloc"]:
            out, _ = fga.fga_reconstruct_points_noalloc(s["beams"], s["eps"], case["tau"], s["xyz"], s["out"],
                                                        precision=p, want_evals=False)
            return _kept(out, case["precision"])
        out, evals = fga.fga_reconstruct_points(s["beams"], s["eps"], case["tau"], s["xyz"], precision=p,
                                                out=s["out"])
        return {"u": _kept(out, case["precision"]), "evals": evals}
    if kind == "grid":
        out, evals = fga.fga_reconstruct_grid(s["beams"], s["eps"], case["tau"], s["mesh"],
                                              precision=PRECISION[case["precision"]], out=s["out"], ws=s["ws"])
        return {"u": _kept(out, case["precision"]), "evals": evals}
    b = s["beams"]
    if kind == "decompose":
        fga.fga_decompose(s["medium"], s["mesh"], s["f"], s["g"], beams=b, ws=s["ws"])
        return {"beams": _parts(b.f64[:, :b.count]), "i32": b.i32[:, :b.count], "lineage": b.lineage[:b.count]}
    if kind in ("homog", "window"):
        fga.fga_decompose(s["medium"], s["mesh"], s["f"], beams=b, ws=s["ws"])
    else:
        fga.fga_decompose_point_source(s["medium"], s["src"], beams=b)
    seis, st = fga.fga_evolve(s["medium"], b, s["dt"], case["steps"], receivers=s["rec"], eps=s["eps"],
                              stride=s["stride"], seis=s.get("seis"), ws=s["ews"], coords=s["coords"],
                              precision=PRECISION[case.get("precision", "fp64")],
                              s_vector=case.get("s_vector", False))
    if kind == "homog":
        out, evals = fga.fga_reconstruct_grid(b, s["eps"], 25.0, s["grid"])
        return {"u": out, "evals": evals, "beams": _by_lineage(b)}
    r = {} if seis is None else {"seis": _kept(seis, case.get("precision", "fp64"))}
    if kind in ("layered", "crosswell"):   # how many beams the interfaces left
        r["info"] = b.info()
    elif kind == "source" or seis is None:
        r["beams"] = _by_lineage(b)
    r.update({k: st[k] for k in ("beam_steps", "evals", "crossings", "spawned", "capped")})
    return r


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _reach(eps, tau, spread):
    """Expected share of uniform points of [0, 1] within the window of a centre 0.5 + spread * normal."""
    r = math.sqrt(2.0 * tau * eps)
    return min(1.0, 2.0 * r * 0.95) ** 3 if spread < 0.5 else min(1.0, r) ** 3


TERM, STEP = 60.0, 4000.0    # flops of a (beam, receiver) term and of a beam's RK4 step in a gridded medium
BEAM = 444.0                 # bytes of a beam's state


def work(case):
    kind = case["kind"]
    if kind == "serve":
        beams = sum(2 * 2 * SWEEP[5 + k % 2][0] ** 3 * SWEEP[5 + k % 2][1] * SWEEP[5 + k % 2][2]
                    for k in range(case["requests"]))
        terms = beams * case["steps"] * 576 * 0.7
        return {"bytes": 2 * BEAM * beams + case["requests"] * 576 * case["steps"] * 48 + 64 ** 3 * 136,
                "flops": beams * case["steps"] * STEP + terms * TERM}
    eps = 2.0 ** -case["log2ieps"]
    if kind in ("points", "grid"):
        n = case["points"] if kind == "points" else case["nx"] * case["ny"] * case["nz"]
        terms = case["beams"] * n * _reach(eps, case["tau"], math.sqrt(0.01 + eps))
        return {"bytes": case["beams"] * 150.0 + n * (72.0 if kind == "points" else 48.0),
                "flops": terms * (TERM if kind == "points" else 24.0)}
    steps, nrec = case.get("steps", 0), case.get("receivers", 0)
    if kind in ("homog", "decompose", "window"):
        ways = 2 if kind == "decompose" else 1
        beams = case["nq"] ** 3 * case["np"] ** 3 * (2 if case.get("merge", True) else 3) * ways
        na, ny = case["nq"] * case["np"], case["ny"]
        fbi = 8.0 * 3 * (ny ** 3 * na + ny ** 2 * na ** 2 + ny * na ** 3) * (3 if ways == 2 else 1)
        inputs = 48.0 * ny ** 3 * ways
        if kind == "decompose":
            return {"bytes": inputs + BEAM * beams, "flops": fbi}
        if kind == "homog":
            pts = case["nout"] ** 3
            return {"bytes": inputs + 3 * BEAM * beams + 48.0 * pts,
                    "flops": fbi + beams * steps * 1647.0 + 24.0 * beams * pts * _reach(eps, 25.0, 0.2)}
        return {"bytes": inputs + 3 * BEAM * beams + 136.0 * case["nmed"] ** 3 + 48.0 * nrec * steps,
                "flops": fbi + beams * steps * STEP + TERM * beams * steps * nrec * _reach(eps, 25.0, 0.2) * 0.4}
    beams = 2 * (2 if case.get("merge", True) else 3) * case["nq"] ** 3 * case["ndir"] * case["nshell"]
    samples = steps // case.get("stride", 1)
    step = {"source": STEP, "layered": 1647.0, "crosswell": STEP}[kind]
    reach = {"source": _reach(eps, 25.0, 0.2) * 0.6, "layered": 0.02, "crosswell": 0.3}[kind]
    return {"bytes": 3 * BEAM * beams + 48.0 * nrec * samples + (136.0 * case["nmed"] ** 3 if kind == "source" else 0),
            "flops": beams * steps * step + TERM * beams * samples * nrec * reach}


# ---------------------------------------------------------------------------
# the same in plain 64-bit torch
# ---------------------------------------------------------------------------

def _dot(a, b):
    return (a * b).sum(-1)


def _frame(P, e):
    sh = torch.linalg.cross(e, P)
    sh = sh / sh.norm(dim=-1, keepdim=True)
    return sh, torch.linalg.cross(P / P.norm(dim=-1, keepdim=True), sh)


def _polarised(b):
    """A (N, 3) complex: a_P P/|P|, or a_SV N_SV + a_SH N_SH (b["A"] where it is advanced itself)."""
    ph = (b["P"] / b["P"].norm(dim=1, keepdim=True)).to(torch.complex128)
    sh, sv = _frame(b["P"], b["e"])
    A = b["a"][:, :1] * sv + b["a"][:, 1:] * sh if b.get("A") is None else b["A"]
    return torch.where((b["branch"] == 0)[:, None], b["a"][:, :1] * ph, A)


def _from_planes(f, i):
    c = lambda k: torch.complex(f[k], f[k + 1])  # noqa: E731
    return {"Q": f[0:3].T, "P": f[3:6].T, "a": torch.stack([c(fga.FGA_A0_RE), c(fga.FGA_A1_RE)], 1), "S": f[fga.FGA_S],
            "w": c(fga.FGA_W_RE), "e": f[fga.FGA_E:fga.FGA_E + 3].T, "branch": i[fga.FGA_BRANCH]}


def _sum_points(b, x, eps, tau):
    R = math.sqrt(2.0 * tau * eps)
    B = (b["w"] * torch.exp(1j * b["S"] / eps))[:, None] * _polarised(b)
    u = torch.zeros((x.shape[0], 3), dtype=torch.complex128, device=x.device)
    per = max(1, 20000000 // max(1, x.shape[0]))
    for k in range(0, B.shape[0], per):
        Q, P = b["Q"][k:k + per], b["P"][k:k + per]
        g, ph, inside = 0.0, 0.0, True
        for d in range(3):
            t = x[:, d, None] - Q[None, :, d]
            g, ph, inside = g + t * t, ph + t * P[None, :, d], inside & (t.abs() <= R)
        u += torch.polar(torch.exp(-g / (2.0 * eps)) * inside, ph / eps) @ B[k:k + per]
    return u


def _sum_grid(b, mesh, eps, tau):
    R = math.sqrt(2.0 * tau * eps)
    B = (b["w"] * torch.exp(1j * b["S"] / eps))[:, None] * _polarised(b)
    n = mesh.n
    u = torch.zeros((3 * n[2], n[1] * n[0]), dtype=torch.complex128, device=_device())
    per = max(64, int(1.5e8 / (n[0] * n[1])))
    for k in range(0, B.shape[0], per):
        E = []
        for d in range(3):
            t = _axis(mesh, d)[None, :] - b["Q"][k:k + per, d, None]
            E.append(torch.polar(torch.exp(-t * t / (2.0 * eps)) * (t.abs() <= R), t * b["P"][k:k + per, d, None] / eps))
        left = (B[k:k + per, :, None] * E[2][:, None, :]).reshape(-1, 3 * n[2])
        u += left.T.contiguous() @ (E[1][:, :, None] * E[0][:, None, :]).reshape(-1, n[1] * n[0])
    return torch.view_as_real(u.reshape(3, n[2], n[1], n[0]).contiguous())


class _Grid:
    """Speeds of a periodic node grid: (c, grad, Hess) for the branch of each beam."""

    def __init__(self, case, seed):
        self.smooth, self.n = case.get("smooth", False), case["nmed"]
        cp, cs = _fields(case, seed)
        self.tab = [self.table(v) for v in ([cp] if cs is None else [cp, cs])]

    def table(self, c):
        n = self.n
        if self.smooth:
            k = (4.0 + 2.0 * torch.cos(2.0 * math.pi * torch.arange(n, dtype=torch.float64, device=c.device) / n)) / 6.0
            return torch.fft.ifftn(torch.fft.fftn(c) / (k[:, None, None] * k[None, :, None] * k[None, None, :])).real
        at = lambda *s: torch.roll(c, [-v for v in s], (2, 1, 0))  # noqa: E731
        one = [(1, 0, 0), (0, 1, 0), (0, 0, 1)]
        f = [c] + [(at(*s) - at(*[-v for v in s])) * (n / 2.0) for s in one]
        f += [(at(*s) - 2.0 * c + at(*[-v for v in s])) * float(n * n) for s in one]
        for s, t in ((0, 1), (0, 2), (1, 2)):
            sg = lambda a, b: at(*[a * one[s][d] + b * one[t][d] for d in range(3)])  # noqa: E731
            f.append((sg(1, 1) - sg(1, -1) - sg(-1, 1) + sg(-1, -1)) * (n * n / 4.0))
        return torch.stack(f, -1)

    def __call__(self, x, S):
        n = self.n
        u = x * n
        i = u.floor()
        t = u - i
        i = i.to(torch.int64)
        out = []
        for tab in self.tab:
            v = torch.zeros((x.shape[0], 10), dtype=torch.float64, device=x.device)
            if self.smooth:
                s = 1.0 - t
                w = torch.stack([s ** 3, 3 * t ** 3 - 6 * t ** 2 + 4, -3 * t ** 3 + 3 * t ** 2 + 3 * t + 1, t ** 3], -1) / 6.0
                d1 = torch.stack([-0.5 * s * s, 1.5 * t * t - 2 * t, -1.5 * t * t + t + 0.5, 0.5 * t * t], -1) * n
                d2 = torch.stack([s, 3 * t - 2, 1 - 3 * t, t], -1) * float(n * n)
                for c in range(64):
                    a, b, d = c & 3, (c >> 2) & 3, c >> 4
                    q = tab[(i[:, 2] - 1 + d) % n, (i[:, 1] - 1 + b) % n, (i[:, 0] - 1 + a) % n]
                    X, Y, Z = [(w[:, m, k], d1[:, m, k], d2[:, m, k]) for m, k in ((0, a), (1, b), (2, d))]
                    for f, (k, l, m) in enumerate(((0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (2, 0, 0), (0, 2, 0),
                                                   (0, 0, 2), (1, 1, 0), (1, 0, 1), (0, 1, 1))):
                        v[:, f] += X[k] * Y[l] * Z[m] * q
            else:
                for c in range(8):
                    o = [c & 1, (c >> 1) & 1, c >> 2]
                    w = 1.0
                    for d in range(3):
                        w = w * (t[:, d] if o[d] else 1.0 - t[:, d])
                    v += w[:, None] * tab[(i[:, 2] + o[2]) % n, (i[:, 1] + o[1]) % n, (i[:, 0] + o[0]) % n]
            out.append(v)
        v = torch.where(S[:, None], out[1] if len(out) > 1 else out[0] / SQRT3, out[0])
        H = torch.stack([v[:, [4, 7, 8]], v[:, [7, 5, 9]], v[:, [8, 9, 6]]], 1)
        return v[:, 0], v[:, 1:4], H


def _homogeneous(x, S):
    c = torch.full((x.shape[0],), SQRT3, dtype=torch.float64, device=x.device)
    c[S] = 1.0
    return c, torch.zeros_like(x), torch.zeros((x.shape[0], 3, 3), dtype=torch.float64, device=x.device)


def _rates(med, b, y, S, sg, vector):
    """Right-hand side of eq:char, eq:DzDt and the amplitude equations."""
    c, g, H = med(y["Q"], S)
    P = y["P"]
    pn = P.norm(dim=1)
    ph = P / pn[:, None]
    r = {"Q": (sg * c)[:, None] * ph, "P": -(sg * pn)[:, None] * g}
    r["S"] = _dot(P, r["Q"]) - sg * c * pn
    cx = lambda v: v.to(torch.complex128)  # noqa: E731
    zg, zp = (y["ZQ"] * cx(g)[:, None, :]).sum(-1), (y["ZP"] * cx(ph)[:, None, :]).sum(-1)
    hz = torch.matmul(y["ZQ"], cx(H).contiguous())
    r["ZQ"] = sg[:, None, None] * (zg[:, :, None] * ph[:, None, :] + (c / pn)[:, None, None] * (y["ZP"] - zp[:, :, None] * ph[:, None, :]))
    r["ZP"] = -sg[:, None, None] * (pn[:, None, None] * hz + zp[:, :, None] * g[:, None, :])
    Z, dZ = y["ZQ"] + 1j * y["ZP"], r["ZQ"] + 1j * r["ZP"]
    cof = torch.stack([torch.linalg.cross(Z[:, (k + 1) % 3], Z[:, (k + 2) % 3]) for k in range(3)], 1)
    tr = (cof * dZ).sum((1, 2)) / (Z[:, 0] * cof[:, 0]).sum(1)
    s = sg * _dot(g, ph) + 0.5 * tr
    if vector:
        dp = -sg[:, None] * g
        dp = dp - ph * _dot(ph, dp)[:, None]
        r["A"] = s[:, None] * y["A"] - (y["A"] * dp).sum(1, keepdim=True) * ph
    ex = torch.linalg.cross(b["e"], P)
    om = torch.where(S, sg * _dot(P, b["e"]) * _dot(b["e"], torch.linalg.cross(g, P)) / _dot(ex, ex), 0.0)
    a0, a1 = y["a"][:, 0], y["a"][:, 1]
    r["a"] = torch.stack([s * a0 - om * a1, torch.where(S, s * a1 + om * a0, 0.0)], 1)
    return r


def _rk4(med, b, dt, vector):
    S, sg = b["branch"] != 0, b["sigma"]
    keys = ["Q", "P", "ZQ", "ZP", "a", "S"] + (["A"] if vector else [])
    y0 = {k: b[k] for k in keys}
    k1 = _rates(med, b, y0, S, sg, vector)
    at = lambda k, h: {n: y0[n] + h * k[n] for n in keys}  # noqa: E731
    k2 = _rates(med, b, at(k1, 0.5 * dt), S, sg, vector)
    k3 = _rates(med, b, at(k2, 0.5 * dt), S, sg, vector)
    k4 = _rates(med, b, at(k3, dt), S, sg, vector)
    for n in keys:
        b[n] = y0[n] + dt / 6.0 * (k1[n] + 2.0 * k2[n] + 2.0 * k3[n] + k4[n])
    if vector:
        ph = b["P"] / b["P"].norm(dim=1, keepdim=True)
        b["A"] = b["A"] - (b["A"] * ph).sum(1, keepdim=True) * ph
    else:
        _reframe(b, S)


def _reframe(b, S):
    """An S beam whose P is within 10 degrees of its frame axis takes the other axis (e_z <-> e_x)."""
    near = S & (_dot(b["P"], b["e"]).abs() / b["P"].norm(dim=1) > math.cos(math.radians(10.0)))
    if not bool(near.any()):
        return
    A = _polarised(b)
    z = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device=b["e"].device)
    was_z = (b["e"] == z).all(1)
    e = torch.where(was_z[:, None], z.flip(0), z)
    b["e"] = torch.where(near[:, None], e, b["e"])
    sh, sv = _frame(b["P"], b["e"])
    a = torch.stack([(A * sv).sum(1), (A * sh).sum(1)], 1)
    b["a"] = torch.where(near[:, None], a, b["a"])


def _planes(b):
    """The 52 planes of a beam set, lineage order."""
    n = b["Q"].shape[0]
    if b.get("A") is not None:   # back to the frame
        S = b["branch"] != 0
        A = b["A"]
        near = S & (_dot(b["P"], b["e"]).abs() / b["P"].norm(dim=1) > math.cos(math.radians(10.0)))
        z = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device=A.device)
        b["e"] = torch.where(near[:, None], torch.where((b["e"] == z).all(1)[:, None], z.flip(0), z), b["e"])
        sh, sv = _frame(b["P"], b["e"])
        b["a"] = torch.where(S[:, None], torch.stack([(A * sv).sum(1), (A * sh).sum(1)], 1), b["a"])
    ZQ, ZP = b["ZQ"].reshape(n, 9).T, b["ZP"].reshape(n, 9).T
    rows = [b["Q"].T, b["P"].T, ZQ.real, ZQ.imag, ZP.real, ZP.imag, torch.view_as_real(b["a"]).reshape(n, 4).T,
            b["S"][None], torch.view_as_real(b["w"]).T, b["e"].T]
    return _parts(torch.cat(rows, 0))


def _new_beams(q, p, e, branch, sigma, w, a):
    n, dev = q.shape[0], q.device
    eye = torch.eye(3, dtype=torch.complex128, device=dev).expand(n, 3, 3)
    return {"Q": q, "P": p, "e": e, "branch": branch, "sigma": sigma, "w": w, "a": a, "ZQ": eye.clone(),
            "ZP": -1j * eye, "S": torch.zeros(n, dtype=torch.float64, device=dev)}


def _axis_of(p):
    near = (p[:, 2].abs() / p.norm(dim=1)) > math.cos(math.radians(20.0))
    z = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device=p.device)
    return torch.where(near[:, None], z.flip(0), z)


def _make_beams(q, p, psi_of, dirs, norm, merge, cull):
    """Beams of the candidates in lineage order; psi_of(branch, sigma, p, n) over the (p, q) pairs; norm per
    branch and pair."""
    out = []
    e = _axis_of(p)
    sh, sv = _frame(p, e)
    for br in ((0, 1) if merge else (0, 1, 2)):
        n = [p / p.norm(dim=1, keepdim=True), sh, sv][br] if not isinstance(p, list) else None
        for sg in dirs:
            psi = psi_of(br, sg, n)
            keep = ~(psi.abs() < cull)
            w = psi * norm
            one, zero = torch.full_like(w, 2.0 ** 1.5), torch.zeros_like(w)
            a = torch.stack([zero, one] if br == 1 else [one, zero], 1)
            if merge and br == 1:
                psv = psi_of(2, sg, sv)
                ksv = ~(psv.abs() < cull)
                a = 2.0 ** 1.5 * torch.stack([torch.where(ksv, psv * norm, 0.0), torch.where(keep, w, 0.0)], 1)
                w, keep = torch.ones_like(w), keep | ksv
            full = lambda v: torch.full((q.shape[0],), v, device=q.device)  # noqa: E731
            b = _new_beams(q, p, e, full(br), full(float(sg)).to(torch.float64), w, a)
            out.append({k: v[keep] for k, v in b.items()})
    return {k: torch.cat([b[k] for b in out]) for k in out[0]}


def _exact_packet(case, seed):
    """The decomposition of the packet cases by three mode products."""
    eps, kind = 2.0 ** -case["log2ieps"], case["kind"]
    y, qm, pm = _cells(case["ny"], 0.0, 1.0), _cells(case["nq"], 0.0, 1.0), _p_mesh(eps, case["np"])
    K = []
    for d in range(3):
        q, p, yy = _axis(qm, d), _axis(pm, d), _axis(y, d)
        t = yy[None, None, :] - q[:, None, None]
        K.append(torch.polar(y.h[d] * torch.exp(-t * t / (2.0 * eps)).expand(-1, case["np"], -1).contiguous(),
                             -p[None, :, None] * t / eps).reshape(-1, case["ny"]))

    def fbi(f):
        t = f.reshape(-1, case["ny"]) @ K[0].T.contiguous()
        t = t.reshape(3, case["ny"], case["ny"], -1).permute(0, 1, 3, 2).contiguous().reshape(-1, case["ny"]) @ K[1].T.contiguous()
        t = t.reshape(3, case["ny"], K[0].shape[0], K[1].shape[0]).permute(0, 2, 3, 1).contiguous()
        t = (t.reshape(-1, case["ny"]) @ K[2].T.contiguous()).reshape(3, case["nq"], case["np"], case["nq"], case["np"], case["nq"], case["np"])
        # (c, qx, px, qy, py, qz, pz) -> (c, pz, py, px, qz, qy, qx)
        return t.permute(0, 6, 4, 2, 5, 3, 1).reshape(3, -1)

    two = kind == "decompose"
    F = fbi(_packet(y, eps, seed, 10))
    G = None
    if two:
        med = _Grid(case, seed)
        g = _packet(y, eps, seed, 11) / eps
        z, yy, x = torch.meshgrid(_axis(y, 2), _axis(y, 1), _axis(y, 0), indexing="ij")
        pts = torch.stack([x.ravel(), yy.ravel(), z.ravel()], 1)
        G = [fbi(g / med(pts, torch.full((pts.shape[0],), s, device=pts.device))[0].reshape(1, *x.shape)) for s in (False, True)]
    grid = lambda m: torch.stack([v.ravel() for v in torch.meshgrid(_axis(m, 2), _axis(m, 1), _axis(m, 0), indexing="ij")][::-1], 1)  # noqa: E731
    qs, ps = grid(qm), grid(pm)
    q, p = qs.repeat(ps.shape[0], 1), ps.repeat_interleave(qs.shape[0], 0)
    pn = p.norm(dim=1)

    def psi(br, sg, n):
        f = (F * n.T).sum(0)
        if not two:
            return f
        return 0.5 * f + sg * 1j * eps / (2.0 * pn) * (G[0 if br == 0 else 1] * n.T).sum(0)

    norm = qm.h[0] ** 3 * pm.h[0] ** 3 * (2.0 * math.pi * eps) ** -4.5
    return _make_beams(q, p, psi, (1, -1) if two else (1,), norm, case.get("merge", True),
                       _cull(case))


def _legendre(n):
    """Gauss-Legendre nodes and weights on [-1, 1], largest first (Golub-Welsch)."""
    k = torch.arange(1, n, dtype=torch.float64)
    b = k / torch.sqrt(4.0 * k * k - 1.0)
    v, V = torch.linalg.eigh(torch.diag(b, 1) + torch.diag(b, -1))
    return v.flip(0).to(_device()), (2.0 * V[0] ** 2).flip(0).to(_device())


def _exact_source(med, spec):
    """A point moment-tensor source with its Ricker weights: closed-form weights of every candidate."""
    eps, nq, ndir, nsh = spec["eps"], spec["nq"], spec["ndir"], spec["nshell"]
    dev = _device()
    x0 = torch.tensor([spec["x0"]], dtype=torch.float64, device=dev)
    xx, yy, zz, xy, xz, yz = spec["M"]
    M = torch.tensor([[xx, xy, xz], [xy, yy, yz], [xz, yz, zz]], dtype=torch.complex128, device=dev)
    half = 4.0 * math.sqrt(eps)
    off = -half + (torch.arange(nq, dtype=torch.float64, device=dev) + 0.5) * (2.0 * half / nq)
    qs = torch.stack([v.ravel() for v in torch.meshgrid(off, off, off, indexing="ij")][::-1], 1) + x0
    t, gw = _legendre(nsh)
    j = torch.arange(ndir, dtype=torch.float64, device=dev)
    z = 1.0 - (2.0 * j + 1.0) / ndir
    r, az = torch.sqrt((1.0 - z * z).clamp(min=0.0)), math.pi * (3.0 - math.sqrt(5.0)) * j
    dirs = torch.stack([r * torch.cos(az), r * torch.sin(az), z], 1)
    cP = med(x0, torch.zeros(1, dtype=torch.bool, device=dev))[0]
    parts = []
    for br in ((0, 1) if spec["merge_s"] else (0, 1, 2)):
        c, g, _ = med(x0, torch.full((1,), br != 0, device=dev))
        lo, hi = 0.2 * cP / c, 2.5 * cP / c
        pn = 0.5 * (lo + hi) + 0.5 * (hi - lo) * t
        dp = (pn ** 2 * 0.5 * (hi - lo) * gw * 4.0 * math.pi / ndir).repeat_interleave(ndir * nq ** 3)
        p = (pn[:, None, None] * dirs[None]).reshape(-1, 3).repeat_interleave(nq ** 3, 0)
        q = qs.repeat(nsh * ndir, 1)
        pm = p.norm(dim=1)
        d = x0 - q
        K = torch.polar(torch.exp(-_dot(d, d) / (2.0 * eps)), -_dot(p, d) / eps)
        grad = K[:, None] * ((-1j * p - d) / eps / c - g / (c * c))
        Mg = grad @ M.T.contiguous()
        x = (c * pm / cP) ** 2
        f = eps / (2.0 * pm) * x * torch.exp(1.0 - x)
        norm = (2.0 * half / nq) ** 3 * dp * (2.0 * math.pi * eps) ** -4.5
        psi = lambda _, sg, n: sg * 1j * f * (Mg * n).sum(1)  # noqa: E731
        b = _make_beams(q, p, psi, (1, -1), norm, spec["merge_s"], 0.0)
        parts.append({k: v[b["branch"] == br] for k, v in b.items()})
    return {k: torch.cat([b[k] for b in parts]) for k in parts[0]}


def _exact_evolve(med, b, dt, steps, rec, stride, eps, vector):
    if vector:
        b["A"] = _polarised(b)
    seis = []
    for k in range(steps):
        _rk4(med, b, dt, vector)
        if rec is not None and (k + 1) % stride == 0:
            seis.append(torch.view_as_real(_sum_points(b, rec, eps, 25.0)))
    return torch.stack(seis, 1) if seis else None


def exact(case, seed):
    kind = case["kind"]
    if kind in ("layered", "crosswell"):
        return None     # interface splitting has no short form
    if kind == "serve":
        med = _Grid(dict(nmed=64), seed)
        out = []
        for r in _requests(case, seed):
            x = r.pop("receivers")
            if 4 * r["nq"] ** 3 * r["ndir"] * r["nshell"] * case["steps"] > 1.2e7:
                out.append(None)    # the larger requests take too long here
                continue
            s = _exact_evolve(med, _exact_source(med, r), 2e-3, case["steps"], x, 1, r["eps"], False)
            out.append(torch.view_as_complex(s).cpu().numpy())
        return out
    eps = 2.0 ** -case["log2ieps"]
    if kind in ("points", "grid"):
        b = _from_planes(*_beam_planes(case, seed))
        if kind == "points":
            u = torch.view_as_real(_sum_points(b, _uniform(_gen(seed, 3), case["points"], 3), eps, case["tau"]))
            return u if case["noalloc"] else {"u": u, "evals": None}
        if 8.0 * 3 * case["beams"] * case["nx"] * case["ny"] * case["nz"] > 5.0e14:
            return None
        return {"u": _sum_grid(b, _grid_mesh(case), eps, case["tau"]), "evals": None}
    steps = case.get("steps", 0)
    if kind == "source":
        if 6.0 * case["nq"] ** 3 * case["ndir"] * case["nshell"] * steps * (4 if case["smooth"] else 1) > 1.2e8:
            return None
        med = _Grid(case, seed)
        b = _exact_source(med, _source_spec(case, seed))
        s = _exact_evolve(med, b, 1e-3, steps, _receivers(case, seed), case["stride"], eps, case["s_vector"])
        return {"seis": s, "beams": _planes(b)}
    if case["nq"] ** 3 * case["np"] ** 3 > 8000000 or (kind == "window" and case["nq"] ** 3 * case["np"] ** 3 * steps > 3e7):
        return None
    b = _exact_packet(case, seed)
    if kind == "decompose":
        return {"beams": _planes(b), "i32": None, "lineage": None}
    if kind == "homog":
        _exact_evolve(_homogeneous, b, 0.005, steps, None, 1, eps, False)
        return {"u": _sum_grid(b, _cells(case["nout"], 0.0, 1.0), eps, 25.0), "evals": None, "beams": _planes(b)}
    rec = _receivers(case, seed) if case["receivers"] else None
    s = _exact_evolve(_Grid(case, seed), b, 1e-3, steps, rec, 1, eps, False)
    return {"beams": _planes(b)} if s is None else {"seis": s}

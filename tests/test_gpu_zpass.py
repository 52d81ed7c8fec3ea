"""The z pass on every padded length, family, precision and schedule, with the
occupied planes at their limits, against the CPU oracle (plan lengths: a body
that does not fill its box is transformed at a shorter length than the grid's
unless the caller fixed the length).

Bars: those of the apply, 1e-12 (FP64) and 2e-5 (FP32) of the term scale.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_1809_00845_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = {B.FP64: 1e-12, B.FP32: 2e-5}
KIND = {B.LAPLACE3D: O.LAPLACE3D, B.NAVIER3D: O.NAVIER3D}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()
    return torch.device("cuda:0")


class _Nodes:
    """m random nodes of an (nx, ny, nz) grid on the planes [lo, hi], both occupied."""

    def __init__(self, n, lo, hi, m=60, seed=0):
        rng = np.random.default_rng(seed)
        z = rng.integers(lo, hi + 1, m)
        z[0], z[1] = lo, hi
        gi = np.stack([rng.integers(0, n[0], m), rng.integers(0, n[1], m), z], 1)
        self.dim, self.n, self.h, self.origin = 3, n, 1.0 / max(n), (0.0, 0.0, 0.0)
        self.nodes = gi * self.h
        nv = rng.normal(size=(m, 3))
        self.normals = nv / np.linalg.norm(nv, axis=1, keepdims=True)
        self.weights = rng.uniform(0.2, 1.5, m) * self.h ** 2


def _check(dev, g, kernel, prec, **kw):
    nc = 3 if kernel == B.NAVIER3D else 1
    m = len(g.weights)
    rng = np.random.default_rng(7)
    q, u = rng.uniform(-1, 1, (nc, m)), rng.uniform(-1, 1, (nc, m))
    plan = B.Plan(g, kernel, precision=prec, nu=0.3, mu=1.0, **kw)
    t = lambda a: torch.tensor(a, device=dev)
    # a first apply on other data: nothing of it may reach the second one
    plan.apply(t(1e3 * u), t(1e3 * q))
    r = plan.apply(t(q), t(u)).cpu().numpy().reshape(nc, m)
    info = dict(plan.info(), lengths=plan.lengths())
    plan.close()
    p = O.problem(g, KIND[kernel], 0.3, 1.0)
    ref, sc = O.apply(p, q if nc > 1 else q[0], u if nc > 1 else u[0], with_scale=True)
    err = np.abs(r - np.reshape(ref, (nc, -1))).max() / np.max(sc)
    assert err < TOL[prec], (kernel, prec, kw, err)
    return info


@pytest.mark.parametrize("pz", [32, 64, 96, 128, 192, 256, 320, 384, 512])
@pytest.mark.parametrize("kernel", [B.LAPLACE3D, B.NAVIER3D])
def test_every_length_with_full_pencils(dev, pz, kernel):
    """All P/2 planes of the grid occupied from first to last (no zero plane
    inside the half pencil), every schedule, the length fixed by the caller."""
    nz = pz // 2
    g = _Nodes((13, 10, nz), 0, nz - 1, seed=pz)
    for prec in (B.FP64, B.FP32):
        for sched in (0, 1, 2) if kernel == B.NAVIER3D and pz in (256, 384, 512) else (0, 1):
            info = _check(dev, g, kernel, prec, pad=(32, 32, pz), autotune=2 + sched)
            assert info["pad"] == info["lengths"] == [32, 32, pz] and info["zsched"] == sched


@pytest.mark.parametrize("lo,hi,nz", [(0, 0, 40), (39, 39, 40), (7, 7, 128), (3, 18, 100), (99, 115, 128), (20, 160, 192), (0, 128, 180),
                                      (10, 57, 128), (1, 96, 128), (60, 200, 256), (0, 127, 256)])
def test_shortened_length(dev, lo, hi, nz):
    """Planes lo..hi of nz: one plane, 2 nzo - 1 just below, at and just above
    a supported length, at either end of the grid; the reported pad stays the
    grid's, the length in use is the smallest for the planes (Navier: not 320)."""
    g = _Nodes((20, 9, nz), lo, hi, seed=lo + hi)
    for kernel in (B.LAPLACE3D, B.NAVIER3D):
        for prec in (B.FP64, B.FP32):
            info = _check(dev, g, kernel, prec)
            want = min(s for s in B.supported_sizes() if s >= 2 * nz)
            assert info["pad"][2] == want and info["z_lo"] == lo and info["z_count"] == hi - lo + 1
            use = min(s for s in B.supported_sizes() if s >= 2 * (hi - lo) + 1)
            use = 384 if use == 320 and kernel == B.NAVIER3D else use
            assert info["lengths"] == info["pad"][:2] + [min(use, want)]


def test_kept_length(dev):
    """A length that the caller asked for is kept, the 16-bit form keeps the grid's,
    2D plans have none along z, Navier's 160-point grid its 320."""
    g = _Nodes((20, 9, 160), 5, 30)
    for prec, kernel, pad, want in ((B.FP64, B.LAPLACE3D, (0, 0, 320), 320), (B.BF16_MFMA, B.LAPLACE3D, (0, 0, 0), 320),
                                    (B.FP32, B.NAVIER3D, (0, 0, 0), 64), (B.FP32, B.LAPLACE3D, (0, 0, 0), 64)):
        plan = B.Plan(g, kernel, precision=prec, pad=pad)
        assert plan.lengths() == [64, 32, want] and plan.info()["pad"] == [64, 32, 320]
        plan.close()
    full = B.Plan(_Nodes((20, 9, 160), 0, 159), B.NAVIER3D, precision=B.FP32)
    assert full.lengths()[2] == 320
    full.close()
    from paper_1809_00845_amd import inputs as I

    flat = B.Plan(I.circle2d(40, 0.4), B.LAPLACE2D)
    assert flat.lengths() == flat.info()["pad"] == [96, 96, 1]
    flat.close()


def test_shortened_length_grid_field_and_batch(dev):
    """The grid evaluation (against the plan with the grid's own length) and
    the batch (bit for bit against the plan) on a shortened plan."""
    g = _Nodes((24, 20, 100), 30, 72, seed=4)
    rng = np.random.default_rng(1)
    q, u = (torch.tensor(rng.uniform(-1, 1, 60), device=dev) for _ in range(2))
    for prec, tol in ((B.FP64, 1e-13), (B.FP32, 1e-5)):
        a = B.Plan(g, B.LAPLACE3D, precision=prec)
        b = B.Plan(g, B.LAPLACE3D, precision=prec, pad=(0, 0, 256))
        fa, fb = a.eval_grid(q, u), b.eval_grid(q, u)
        assert fa.shape == fb.shape == (1, 43, 20, 24)
        assert float((fa - fb).abs().max()) <= tol * float(fb.abs().max())
        batch = B.Batch([a], nrhs=2)
        r = torch.empty(120, dtype=torch.float64, device=dev)
        batch.apply(torch.cat([q, u]), torch.cat([u, q]), r)
        assert torch.equal(r, torch.cat([a.apply(q, u), a.apply(u, q)]))
        batch.close()
        a.close()
        b.close()


# (family, precision, padded lengths, schedule): lengths whose fastest schedule is not
# the others', both sides of the few-pencils rule, and the length without a third one
DEFAULTS = [(B.LAPLACE3D, B.FP64, (32, 32, 384), 1), (B.LAPLACE3D, B.FP64, (32, 32, 320), 0),
            (B.LAPLACE3D, B.FP32, (32, 32, 384), 0), (B.NAVIER3D, B.FP64, (32, 32, 320), 0),
            (B.NAVIER3D, B.FP64, (32, 32, 512), 2), (B.NAVIER3D, B.FP64, (96, 64, 256), 1),
            (B.NAVIER3D, B.FP32, (256, 128, 256), 1),
            (B.NAVIER3D, B.FP32, (256, 192, 256), 0), (B.NAVIER3D, B.FP32, (32, 32, 320), 1)]


@pytest.mark.parametrize("kernel,prec,pad,want", DEFAULTS)
def test_default_schedule(dev, kernel, prec, pad, want):
    """The schedule without autotuning: the measured one of the length, one that
    exists, and the same results as the oracle's."""
    g = _Nodes((13, 10, pad[2] // 2), 0, pad[2] // 2 - 1, seed=pad[2])
    assert _check(dev, g, kernel, prec, pad=pad)["zsched"] == want


@pytest.mark.parametrize("py", [32, 64, 96, 320])
@pytest.mark.parametrize("nz", [1, 2, 15, 16])
def test_short_pencils(dev, py, nz):
    """Laplace at 32 points, four (schedule 0) or eight lanes per pencil: sixteen ky
    of a wavefront on both sides of Py / 2, with one, few and all planes occupied."""
    g = _Nodes((16, py // 2, nz), 0, nz - 1, seed=py + nz)
    for prec in (B.FP64, B.FP32):
        for sched in (0, 1):
            _check(dev, g, B.LAPLACE3D, prec, pad=(32, py, 32), autotune=2 + sched)


@pytest.mark.parametrize("use_graph", [True, False])
@pytest.mark.parametrize("kernel", [B.LAPLACE3D, B.NAVIER3D])
def test_batch_of_lengths(dev, kernel, use_graph):
    """Members of one grid whose bodies occupy different numbers of planes (their z
    passes differ in length and schedule, everything else runs as one group), in an
    order that is not that of the lengths: every member has its plan's bits."""
    spans = [(3, 40), (10, 10), (0, 63), (20, 45), (5, 20), (1, 40)]
    geoms = [_Nodes((24, 20, 64), lo, hi, m=50 + 7 * i, seed=i) for i, (lo, hi) in enumerate(spans)]
    nc = 3 if kernel == B.NAVIER3D else 1
    rng = np.random.default_rng(3)
    for prec in (B.FP64, B.FP32):
        plans = [B.Plan(g, kernel, precision=prec, autotune=2 + i % 2) for i, g in enumerate(geoms)]
        batch = B.Batch(plans, nrhs=2, use_graph=use_graph)
        n = sum(batch.lengths)
        q, u = (torch.tensor(rng.uniform(-1, 1, n), device=dev) for _ in range(2))
        cut = lambda t, k: t[batch.offsets[k]:batch.offsets[k] + batch.lengths[k]].contiguous()
        ref = torch.cat([plans[k // 2].apply(cut(q, k), cut(u, k)) for k in range(len(batch.offsets))])
        assert n == sum(2 * nc * len(g.weights) for g in geoms)
        for _ in range(3):
            r = torch.full_like(q, float("nan"))
            batch.apply(q, u, r)
            assert torch.equal(r, ref)
            _ = (q * 2.0).sum().item()  # eager work between replays
        batch.close()
        for p in plans:
            p.close()


def test_batch_in_branches(dev):
    """Two grids whose intermediates together take 64 to 256 MB (the graph then holds
    the groups as parallel branches): every replay gives the plans' bits."""
    geoms = [_Nodes((48, 48, 48), 2, 40, m=300), _Nodes((64, 64, 64), 5, 50, m=400), _Nodes((48, 40, 48), 0, 47, m=200)]
    plans = [B.Plan(g, B.LAPLACE3D, precision=B.FP64) for g in geoms]
    batch = B.Batch(plans, nrhs=2, use_graph=True)
    rng = np.random.default_rng(8)
    n = sum(batch.lengths)
    cut = lambda t, k: t[batch.offsets[k]:batch.offsets[k] + batch.lengths[k]].contiguous()
    for _ in range(4):  # replays on new inputs, with eager work between them
        q, u = (torch.tensor(rng.uniform(-1, 1, n), device=dev) for _ in range(2))
        r = torch.full_like(q, float("nan"))
        batch.apply(q, u, r)
        assert torch.equal(r, torch.cat([plans[k // 2].apply(cut(q, k), cut(u, k)) for k in range(6)]))
    batch.close()
    for p in plans:
        p.close()


def test_autotune_times_each_schedule_once(dev):
    """Numbers of one schedule share its time (and the first of them is kept): at 64
    points there is one, at 96 there are two, Navier FP64 at 320 has one."""
    for kernel, prec, pz, same in ((B.LAPLACE3D, B.FP32, 64, True), (B.LAPLACE3D, B.FP32, 96, False),
                                   (B.NAVIER3D, B.FP64, 320, True), (B.NAVIER3D, B.FP64, 256, False)):
        g = _Nodes((13, 10, pz // 2), 0, pz // 2 - 1)
        plan = B.Plan(g, kernel, precision=prec, pad=(32, 32, pz), autotune=1)
        info = plan.info()
        plan.close()
        t = info["tune_us"]
        assert (t[0] == t[1]) == same and t[info["zsched"]] == min(x for x in t if x > 0)
        assert not same or info["zsched"] == 0
        if kernel == B.NAVIER3D and pz == 256:
            assert t[2] > 0 and t[2] == t[0]  # 8, 8, 2 in wide tiles: schedule 0's


def test_autotune_cache(dev, tmp_path, monkeypatch):
    """A second plan reads what the first one stored, for either forward width."""
    path = tmp_path / "tune"
    monkeypatch.setenv("BEMFFT_TUNE_CACHE", str(path))
    g = _Nodes((20, 16, 24), 2, 20)
    first = B.Plan(g, B.LAPLACE3D, precision=B.FP32, autotune=1)
    a = first.info()
    first.close()
    key, value = path.read_text().split()
    for stored in range(2):
        for width in (1, 2):
            path.write_text(f"{key} {stored + 4 * (width - 1)}\n")
            plan = B.Plan(g, B.LAPLACE3D, precision=B.FP32, autotune=1)
            b = plan.info()
            plan.close()
            assert (b["zsched"], b["fwd_xg"]) == (stored, width) and not any(b["tune_us"])
    assert int(value) == a["zsched"] + 4 * (a["fwd_xg"] - 1)

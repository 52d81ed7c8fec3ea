"""2D plans at the limits of their kernels' rules: node counts and rows on both
sides of where the fields are folded into the transform kernel (three rows of 24 or
more; 1792 nodes below 512 points along x; three rows of 8 or more beside 1152 other
nodes, in rows of at most two where Py = 1024), where the node sums go wide (4096
nodes, 8192 with three outputs) and where every node lies in a long row (8 or
more, 24 in the folded form); rows of 1 to nx nodes around the sizes where a thread,
a wavefront or an FFT sums them (and several rounds of a wavefront); every padded
length on either axis.  Bars: normwise against the direct sums, 1e-12 in FP64,
2e-5 in FP32, as for ordinary geometries: they grow with log P only."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_1809_00845_amd import binding as B  # noqa: E402
from paper_1809_00845_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = {B.FP64: 1e-12, B.FP32: 2e-5}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()
    return torch.device("cuda:0")


def rows_geometry(nx, ny, counts, seed=0):
    """counts[y] nodes at random x of row y, in shuffled order, random normals."""
    rng = np.random.default_rng(seed)
    pts = [(x, y) for y, c in enumerate(counts) for x in rng.choice(nx, size=c, replace=False)]
    pts = np.asarray(pts, dtype=np.float64)[rng.permutation(len(pts))]
    h = 1.0 / max(nx, ny)
    a = rng.uniform(0, 2 * np.pi, len(pts))
    return I.Geometry(2, (nx, ny, 1), h, (0.0, 0.0, 0.0), pts * h, np.stack([np.cos(a), np.sin(a)], 1),
                      h * rng.uniform(0.5, 1.5, len(pts)), np.array([0.5, 0.5]), f"rows{nx}x{ny}")


def spread(total, rows, ny, most):
    """total nodes over the first 'rows' of ny rows, at most 'most' each."""
    c = [min(most, total // rows + (1 if y < total % rows else 0)) for y in range(rows)]
    assert sum(c) == total
    return c + [0] * (ny - rows)


MIXED = [1, 0, 8, 9, 23, 24, 2, 64, 65, 0, 16, 3]
CASES = {
    # the folded form's limits: long rows, nodes of a short transform
    "long3": (100, 40, [30] * 3 + [2] * 37),
    "long4": (100, 40, [30] * 4 + [2] * 36),
    "m1792": (128, 128, [14] * 128),
    "m1793": (128, 128, [15] + [14] * 127),
    "m4100": (128, 400, [120] + [10] * 398 + [0]),
    # of a longer one: heavy rows, other nodes, rows of two at 1024 points
    "heavy3": (200, 200, [23, 8, 100] + [5] * 197),
    "heavy4": (200, 200, [23, 8, 100, 8] + [5] * 196),
    "heavy4x256": (256, 200, [23, 8, 100, 8] + [5] * 196),
    "m1792x384": (192, 128, [14] * 128),
    "m1793x384": (192, 128, [15] + [14] * 127),
    "light1152": (256, 256, [5] * 128 + [4] * 128),
    "light1153": (256, 256, [5] * 129 + [4] * 127),
    "two1024": (300, 512, [2] * 500 + [0] * 11 + [300]),
    "three1024": (300, 512, [2] * 500 + [3] + [0] * 10 + [300]),
    # rows of 7 and 8 nodes side by side, every row of 8
    "rows78": (512, 256, [7, 8] * 128),
    "rows8": (512, 256, [8] * 256),
    # wide sums: 4096 and 4097 nodes
    "wide4096": (512, 512, [7] * 448 + [15] * 64),
    "wide4097": (512, 512, [7] * 448 + [15] * 63 + [16]),
    # long rows and node counts of several rounds
    "long8": (100, 40, [30] * 8 + [2] * 32),
    "long9": (100, 40, [30] * 9 + [2] * 31),
    "m4096": (250, 250, spread(4096, 250, 250, 23)),
    "m4097": (250, 250, spread(4097, 250, 250, 23)),
    # wide sums: 8192 and 8193 nodes
    "m8192": (400, 390, spread(8192, 390, 390, 23)),
    "m8193": (400, 390, spread(8193, 390, 390, 23)),
    # all nodes in long rows, some rows empty
    "alllong": (300, 30, [0, 24, 299, 300, 0, 25] * 5),
    "onerow": (512, 16, [0] * 7 + [512] + [0] * 8),
    # a wavefront with more heavy rows than it sums itself, and rows of every kind
    "heavy": (128, 128, [9, 20, 10] * 42 + [0, 128]),
    "mixed64": (70, 12, MIXED),
    # every padded length along y (and others along x)
    **{f"ny{n}": (nx, n, (MIXED * 50)[:n]) for n, nx in
       ((15, 66), (31, 500), (45, 130), (64, 200), (96, 96), (127, 160), (150, 66), (191, 256), (256, 320), (512, 90))},
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("kernel", [B.LAPLACE2D, B.HALFSPACE])
def test_flat_rules(dev, name, kernel):
    nx, ny, counts = CASES[name]
    g = rows_geometry(nx, ny, counts, seed=len(name))
    nc = 3 if kernel == B.HALFSPACE else 1
    rng = np.random.default_rng(5)
    q, u = rng.uniform(-1, 1, (nc, g.m)), rng.uniform(-1, 1, (nc, g.m))
    p = O.problem(g, O.HALFSPACE if nc == 3 else O.LAPLACE2D, 0.3, 1.0)
    t1 = min(g.m, 300)
    ref, sc = O.apply(p, q if nc > 1 else q[0], u if nc > 1 else u[0], with_scale=True, targets=(0, t1))
    qd, ud = torch.tensor(q, device=dev), torch.tensor(u, device=dev)
    for prec in (B.FP64, B.FP32):
        plan = B.Plan(g, kernel, precision=prec, nu=0.3, mu=1.0)
        r = plan.apply(qd, ud)
        again = plan.apply(qd, ud)
        assert torch.equal(r, again)
        err = np.abs(r.cpu().numpy().reshape(nc, g.m)[:, :t1] - np.reshape(ref, (nc, -1))).max() / np.max(sc)
        assert err < TOL[prec], (prec, err)
        # the same plan as a member of a batch: the same bits
        batch = B.Batch([plan], nrhs=1, use_graph=False)
        rb = torch.empty_like(r)
        batch.apply(qd.reshape(-1), ud.reshape(-1), rb)
        assert torch.equal(r.reshape(-1), rb.reshape(-1))
        batch.close()
        plan.close()


# right-hand sides on both sides of the blocks that the folded form keeps resident
# (256 CUs of two wavefronts per SIMD: 512 blocks of three or four wavefronts, 2048 of one)
MANY = [("m1792", 3), ("m1792", 4), ("heavy3", 1), ("heavy3", 2), ("two1024", 2), ("light1152", 2), ("long3", 15),
        ("long3", 16), ("mixed64", 33), ("rows78", 3), ("heavy", 5)]


@pytest.mark.parametrize("name,nrhs", MANY)
@pytest.mark.parametrize("kernel", [B.LAPLACE2D, B.HALFSPACE])
def test_batches_of_many_members(dev, name, nrhs, kernel):
    """Batches that fill the chip take the lean form of the transform kernel: every
    member has its plan's bits."""
    nx, ny, counts = CASES[name]
    g = rows_geometry(nx, ny, counts, seed=len(name))
    n = (3 if kernel == B.HALFSPACE else 1) * g.m
    rng = np.random.default_rng(6)
    q, u = (torch.tensor(rng.uniform(-1, 1, (nrhs, n)), device=dev) for _ in range(2))
    for prec in (B.FP64, B.FP32):
        plan = B.Plan(g, kernel, precision=prec, nu=0.3, mu=1.0)
        batch = B.Batch([plan], nrhs=nrhs, use_graph=True)
        ref = torch.stack([plan.apply(q[i], u[i]) for i in range(nrhs)])
        for _ in range(3):
            r = torch.full_like(q, float("nan"))
            batch.apply(q.reshape(-1), u.reshape(-1), r)
            assert torch.equal(r, ref)
            _ = (q * 2.0).sum().item()  # eager work between replays
        batch.close()
        plan.close()

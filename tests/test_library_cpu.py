"""Host-side checks of the C-ABI library that need no GPU: it loads, exports
every function the header declares, and rejects bad arguments before any
device work starts."""

import ctypes
import os
import re

import numpy as np
import pytest

from paper_1809_00845_amd import binding as B
from paper_1809_00845_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    txt = open(os.path.join(ROOT, "include", "bemfft.h")).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b(bemfft_[a-z0-9_]+)\s*\(", txt)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_1809_00845_amd import build

        build.build()
    return B.load()


def test_header_symbols_exported(lib):
    names = _declared()
    assert len(names) >= 10
    for n in names:
        assert hasattr(lib, n), n
    assert set(B.EXPORTS) == set(names)


def test_strerror_and_sizes(lib):
    assert B.strerror(0) == "ok"
    assert "invalid" in B.strerror(B.EINVAL)
    assert B.supported_sizes() == [32, 64, 96, 128, 192, 256, 320, 384, 512, 1024]


def _expect(status_fn, code):
    with pytest.raises(B.BemfftError) as ei:
        status_fn()
    assert ei.value.status == code


def test_plan_validation_rejects_before_device_work(lib):
    g = I.circle2d(32, 0.3)
    # kernel / dimension mismatch
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, g.weights, B.LAPLACE3D), B.EINVAL)
    # node off the grid
    bad = g.nodes.copy()
    bad[3, 0] = 1.5
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, bad, g.normals, g.weights, B.LAPLACE2D), B.EINVAL)
    # non-positive weight
    w = g.weights.copy()
    w[0] = 0.0
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, w, B.LAPLACE2D), B.EINVAL)
    # non-finite coordinate
    nn = g.nodes.copy()
    nn[1, 1] = np.nan
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, nn, g.normals, g.weights, B.LAPLACE2D), B.EINVAL)
    # padded length shorter than 2n - 1 / not a supported length
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, g.weights, B.LAPLACE2D,
                                         pad=(32, 64, 0)), B.EUNSUPPORTED)
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, g.weights, B.LAPLACE2D,
                                         pad=(66, 64, 0)), B.EUNSUPPORTED)
    # Navier material parameters
    s = I.cube3d(16, 8)
    _expect(lambda: B.bemfft_plan_create(3, s.n, s.h, s.nodes, s.normals, s.weights, B.NAVIER3D, nu=0.5),
            B.EINVAL)
    _expect(lambda: B.bemfft_plan_create(3, s.n, s.h, s.nodes, s.normals, s.weights, B.NAVIER3D, mu=0.0),
            B.EINVAL)
    # C_USER without values
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, g.weights, B.LAPLACE2D,
                                         c_mode=B.C_USER), B.EINVAL)
    # half-space: a 2D surface grid, elastic constants checked; normals are optional
    hs = I.halfspace_patch(32, 0.3)
    _expect(lambda: B.bemfft_plan_create(3, s.n, s.h, s.nodes, s.normals, s.weights, B.HALFSPACE), B.EINVAL)
    _expect(lambda: B.bemfft_plan_create(2, hs.n, hs.h, hs.nodes, None, None, B.HALFSPACE, nu=0.5), B.EINVAL)
    _expect(lambda: B.bemfft_plan_create(2, hs.n, hs.h, hs.nodes, None, None, B.HALFSPACE, mu=-1.0), B.EINVAL)
    # unknown kernel family
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, g.weights, 4), B.EINVAL)
    # NULL normals are refused for the boundary families
    _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, None, g.weights, B.LAPLACE2D), B.EINVAL)
    # grid sizes: 2D up to 512 per axis (P = 1024), 3D up to 256 (P = 512)
    sq = I.square2d(513, 500)
    _expect(lambda: B.bemfft_plan_create(2, sq.n, sq.h, sq.nodes, sq.normals, sq.weights, B.LAPLACE2D), B.EINVAL)
    s3 = I.sphere3d(16, 0.35)
    _expect(lambda: B.bemfft_plan_create(3, (257, 16, 16), s3.h, s3.nodes, s3.normals, s3.weights, B.LAPLACE3D),
            B.EINVAL)
    _expect(lambda: B.bemfft_plan_create(3, s3.n, s3.h, s3.nodes, s3.normals, s3.weights, B.LAPLACE3D,
                                         pad=(1024, 32, 32)), B.EUNSUPPORTED)
    # autotune outside [0, 4]
    for t in (-1, 5):
        _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, g.weights, B.LAPLACE2D,
                                             autotune=t), B.EINVAL)
    # cell rule outside [0, 8]
    for q in (-1, 9):
        _expect(lambda: B.bemfft_plan_create(2, g.n, g.h, g.nodes, g.normals, g.weights, B.LAPLACE2D,
                                             cell_quad=q), B.EINVAL)


def test_null_arguments(lib):
    assert lib.bemfft_apply(None, None, None, None, None) == B.EINVAL
    assert lib.bemfft_solve(None, None, None, None, None, None, None) == B.EINVAL
    assert lib.bemfft_plan_destroy(None) == 0
    assert lib.bemfft_plan_get_info(None, None) == B.EINVAL
    assert lib.bemfft_plan_get_lengths(None, None) == B.EINVAL


def test_net_validation_rejects_before_device_work(lib):
    for grid, layers, dil in [(2, 4, (1, 2, 4, 8)), (300, 4, (1, 2, 4, 8)), (16, 1, (1,)), (16, 2, (1, 0)),
                              (16, 2, (1, 17))]:
        with pytest.raises(B.BemfftError) as ei:
            B.Net(grid, dil[:layers])
        assert ei.value.status == B.EINVAL


def test_node_count_limit(lib):
    """Node counts whose [F][m] field index would overflow 32 bits are refused
    before any node is read (the pointer below holds one node only)."""
    L = lib
    g = B.bemfft_grid()
    g.dim = 3
    for a in range(3):
        g.n[a] = 16
    g.h = 1.0 / 16
    one = np.full(3, 0.5)
    dp = ctypes.POINTER(ctypes.c_double)
    out = ctypes.c_void_p()
    for kernel, fields in ((B.NAVIER3D, 9), (B.LAPLACE3D, 4)):
        m = (2 ** 31 - 1) // fields + 1
        st = L.bemfft_plan_create(ctypes.byref(out), ctypes.byref(g), m, one.ctypes.data_as(dp),
                                  one.ctypes.data_as(dp), None, kernel, 0.3, 1.0, None)
        assert st == B.EINVAL, (kernel, st)
        assert "node count" in B.last_error()
    st = L.bemfft_plan_create(ctypes.byref(out), ctypes.byref(g), 0, one.ctypes.data_as(dp), one.ctypes.data_as(dp),
                              None, B.LAPLACE3D, 0.3, 1.0, None)
    assert st == B.EINVAL


def test_binding_rejects_bad_tensors_before_any_call(lib):
    """The binding checks device, dtype, contiguity and length itself: the
    library trusts the sizes it is given.  CPU tensors, float32 vectors,
    short vectors and a non-uint8 bc raise ValueError without a library
    call (the fake handle would fail loudly if one were made)."""
    torch = pytest.importorskip("torch")
    fake = ctypes.c_void_p(1)
    cpu = torch.zeros(10, dtype=torch.float64)
    with pytest.raises(ValueError, match="GPU"):
        B.bemfft_apply(fake, cpu, cpu, cpu, n=10)
    with pytest.raises(ValueError, match="torch tensor"):
        B.bemfft_apply(fake, np.zeros(10), cpu, cpu, n=10)
    with pytest.raises(ValueError, match="float64"):
        B._f64(torch.zeros(10, dtype=torch.float32), 10, "q")
    with pytest.raises(ValueError, match="elements"):
        B.bemfft_apply(fake, torch.zeros(9, dtype=torch.float64), cpu, cpu, n=10)
    with pytest.raises(ValueError, match="uint8"):
        B._u8(torch.zeros(10, dtype=torch.int32), 10, "bc")
    with pytest.raises(ValueError, match="contiguous"):
        B._ptr(torch.zeros(10, 2, dtype=torch.float64).t())
    with pytest.raises(ValueError, match="GPU"):
        B.bemfft_solve(fake, torch.zeros(10, dtype=torch.uint8), cpu, cpu, n=10)

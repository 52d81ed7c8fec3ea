"""The network's convolution kernels at the edges of their ranges: grids below,
at and above a tile of 16 voxels and a block's 256 positions, and dilations up
to and past the 16 up to which a block's halo is shared (and past the grid's
half, where most taps leave the grid).  Bars as for the same entry points at
ordinary sizes: they are per layer and do not depend on grid or dilation."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import nn_oracle as NN  # noqa: E402
from paper_1809_00845_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu

# (grid, dilations): first, hidden and output layers on both sides of 16
EDGES = [(4, (1, 2, 3, 4)), (6, (6, 5, 1)), (16, (15, 16, 1, 16)), (17, (16, 17, 16, 17)), (20, (17, 16, 18)),
         (33, (16, 17, 8, 16)), (41, (1, 16))]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()
    return torch.device("cuda:0")


def _case(G, dil):
    rng = np.random.default_rng(1000 + G)
    net = B.Net(G, dil, seed=4)
    p = (0.2 * rng.standard_normal(net.nparam)).astype(np.float32)
    net.set_params(p)
    x = rng.standard_normal((6, G ** 3)).astype(np.float32)
    return rng, net, p.astype(np.float64), x


@pytest.mark.parametrize("G,dil", EDGES)
def test_infer_edges(dev, G, dil):
    _, net, p, x = _case(G, dil)
    y = torch.empty(G ** 3, dtype=torch.float32, device=dev)
    net.infer(torch.tensor(x, device=dev), y)
    ref = NN.forward(p, list(dil), x.astype(np.float64).reshape(6, G, G, G))[0].ravel()
    got = y.cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-2 * np.abs(ref).max()
    assert np.linalg.norm(got - ref) <= 3e-3 * np.linalg.norm(ref)
    net.close()


@pytest.mark.parametrize("G,dil", EDGES)
def test_forward_and_gradients_edges(dev, G, dil):
    rng, net, p, x = _case(G, dil)
    xt = torch.tensor(x, device=dev)
    y = torch.empty(G ** 3, dtype=torch.float32, device=dev)
    net.forward(xt, y)
    x3 = x.astype(np.float64).reshape(6, G, G, G)
    ref = NN.forward(p, list(dil), x3)[0].ravel()
    assert np.abs(y.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
    nt = G ** 3 // 3
    vox = rng.choice(G ** 3, size=nt, replace=False).astype(np.int32)
    tgt = rng.standard_normal(nt).astype(np.float32)
    wt = (rng.uniform(0.5, 1.5, nt) / nt).astype(np.float32)
    args = (xt,) + tuple(torch.tensor(a, device=dev) for a in (vox, tgt, wt))
    L, g = net.gradients(*args)
    Lr, gr = NN.loss_and_grad(p, list(dil), x3, vox, tgt.astype(np.float64), wt.astype(np.float64))
    assert abs(L - Lr) <= 1e-5 * abs(Lr)
    assert np.abs(g - gr).max() <= 2e-4 * np.abs(gr).max()
    assert np.linalg.norm(g - gr) <= 2e-5 * np.linalg.norm(gr)
    assert np.array_equal(net.gradients(*args)[1], g)
    net.close()

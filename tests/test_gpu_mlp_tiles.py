"""The regressor's 16-row tiles against the FP64 reference (bars as in test_gpu_mlp): one tile and its neighbours,
the largest batch with one tile per block (1024 tiles) and the first with four, whose last block has rows in one
tile only; widths off the 4 x 4 gradient tiles and above one wave's 64 units."""
import numpy as np
import pytest

from test_gpu_mlp import _data, _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,h", [(16, 20, 64), (17, 5, 33), (16384, 9, 20), (16385, 9, 20), (16400, 33, 65),
                                   (40, 256, 37), (50, 3, 106)])
def test_tiles(n, d, h):
    import paper_2603_07387_amd as T
    from oracle import mlp
    net = T.MLP(d, h, seed=n)
    X, y = _data(n, d, n + 1)
    p = net.params()
    pred = net.predict(_dev(X)).cpu().numpy().astype(np.float64)
    ref = mlp.forward(p, X, d, h)
    assert np.all(np.abs(pred - ref) <= 1e-4 * (1 + np.abs(ref)))
    g, loss = net.grad(_dev(X), _dev(y))
    lref, gref = mlp.loss_and_grad(p, X, y, d, h)
    assert abs(loss - lref) <= 1e-4 * max(lref, 1e-3)
    assert np.linalg.norm(g.cpu().numpy().astype(np.float64) - gref) <= 1e-4 * np.linalg.norm(gref)

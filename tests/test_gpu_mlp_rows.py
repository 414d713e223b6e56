"""Predictions by rows (narrow networks, many rows) against the FP64 reference (bar as in test_gpu_mlp) and, bit for bit,
against the same rows in calls of fewer, which the 16-row tiles take: both sum every dot product in the order of its
index.  Edges: one unit, units off fours, 16 and 32 units, inputs of one, of 32 and around several times 32, a last wave
of one row, the rule's first row count."""
import numpy as np
import pytest

from test_gpu_mlp import _data, _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,h", [(8192, 8, 16), (8193, 32, 13), (16385, 33, 16), (16448, 1, 1), (16400, 65, 32),
                                   (17001, 256, 30), (16385, 31, 17)])
def test_rows(n, d, h):
    import paper_2603_07387_amd as T
    from oracle import mlp
    net = T.MLP(d, h, seed=n)
    X, _ = _data(n, d, n + 1)
    Xd = _dev(X)
    pred = net.predict(Xd).cpu().numpy()
    ref = mlp.forward(net.params(), X, d, h)
    assert np.all(np.abs(pred.astype(np.float64) - ref) <= 1e-4 * (1 + np.abs(ref)))
    parts = [net.predict(Xd[u:u + 4000].contiguous()).cpu().numpy() for u in range(0, n, 4000)]
    assert np.array_equal(pred, np.concatenate(parts))

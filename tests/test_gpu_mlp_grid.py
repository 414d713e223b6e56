"""Predictions of more rows than blocks fit into one row of the grid (2^21 blocks of 64 rows), the last rows against the
same rows in a call of their own, bit for bit: by rows and by tiles."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h", [2, 33])
def test_many_rows(h):
    import torch
    import paper_2603_07387_amd as T
    net = T.MLP(1, h, seed=h)
    n = (1 << 27) + 64 * 5 + 3
    X = torch.randn(n, 1, device="cuda")
    pred = net.predict(X)
    for first, count in ((0, 200), ((1 << 27) - 100, 400), (n - 70, 70)):
        assert torch.equal(pred[first:first + count], net.predict(X[first:first + count].contiguous())), first

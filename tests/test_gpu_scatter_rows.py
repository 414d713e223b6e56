"""Scatter blocks by the rows whose words they hold at a time (2048, 1024 or 512 for one, two or more samples per pass):
slots of as many rows, one more and several times as many, of few and of many hash words, a single column among them.
The sums are exact integers, so every schedule gives the same sketches bit for bit; against the FP64 oracle (bars as in
test_gpu_scatter)."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import TAU, make_plan
from test_gpu_scatter import T  # noqa: F401

pytestmark = pytest.mark.gpu


def networks():
    rng = np.random.default_rng(2)
    out = []
    for shapes, edges in (([(2048, 4), (2048, 4)], [(0, 2), (1, 3)]), ([(2049, 3), (2049, 3)], [(1, 3), (0, 2)]),
                          ([(1025, 5), (1025, 5)], [(0, 2), (1, 3)]), ([(22, 250, 12), (250, 12, 22)], [(3, 1), (4, 2), (5, 0)]),
                          ([(31, 33, 40, 1), (31, 33, 40, 1)], [(0, 4), (5, 1), (2, 6), (7, 3)])):
        data = [rng.choice([-1.0, 1.0], s) * (0.5 + 0.5 * rng.random(s)) for s in shapes]
        out.append(W.Network([len(s) for s in shapes], [n for s in shapes for n in s], edges, data))
    return out


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_rows(T, orc, dtype, monkeypatch):  # noqa: F811
    m, S = 256, 9
    want = None
    for banks in ("1", "2"):
        for sb in ("1", "2", "4", "8"):
            monkeypatch.setenv("TN_SCATTER_BANKS", banks)
            monkeypatch.setenv("TN_SCATTER_SB", sb)
            plan, views = make_plan(T, networks(), dtype, m, S, 40)
            got = plan.sketches(first=0, count=S).cpu().numpy()
            want = got if want is None else want
            assert np.array_equal(got, want), (banks, sb)
    k0 = 0
    for j, net in enumerate(views):
        absnet = net.with_data([np.abs(x) for x in net.data])
        for r in (0, S - 1):
            ref = orc.m1_estimate(net, m, 40 + j, r, combine="dft", want_sketches=True)["sketches"]
            tables = []
            for e in range(net.t):
                h, _ = orc.hash_table(40 + j, r, e, net.dims[net.edges[e][0]], m)
                tables.append(np.concatenate([h, np.ones_like(h)]))
            A = orc.m1_estimate(absnet, m, 0, 0, tables=tables, combine="dft", want_sketches=True)["sketches"]
            err = np.abs(want[r, k0:k0 + net.p] - ref)
            assert np.all(err <= TAU[dtype] * A + 1e-300), (j, r, (err - TAU[dtype] * A).max())
        k0 += net.p

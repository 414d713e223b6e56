"""Sketches of FP64 entries up to the type's largest: the fixed-point scale of entries from 2^1023 on, when a block finds
the largest entry itself and when a later chunk of samples takes the recorded bound.  Against the FP64 oracle, bucket by
bucket (bars as in test_gpu_scatter; the entries' sums stay below 2^1024)."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import TAU, make_plan
from test_gpu_scatter import T  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [31, 33])  # one wave per sample, a block
@pytest.mark.parametrize("m, S, samples", [(64, 3, [0, 1, 2]), (2, 65600, [0, 65534, 65599])])
def test_largest_entries(T, orc, n, m, S, samples):  # noqa: F811
    rng = np.random.default_rng(n)
    data = []
    for _ in range(2):
        x = np.ldexp(rng.choice([-1.0, 1.0], (n, n)) * (1 + rng.random((n, n))), 1012)
        x[n // 2, 3] = np.ldexp(1.75, 1023)
        data.append(x)
    net = W.Network([2, 2], [n] * 4, [(0, 3), (1, 2)], data)
    plan, views = make_plan(T, [net], "float64", m, S, 40)
    if S > 65535:
        assert plan.query(9) < S  # more than one chunk
    got = plan.sketches(first=0, count=S)
    absnet = views[0].with_data([np.abs(x) for x in views[0].data])
    for r in samples:
        ref = orc.m1_estimate(views[0], m, 40, r, combine="dft", want_sketches=True)["sketches"]
        tables = []
        for e in range(net.t):
            h, _ = orc.hash_table(40, r, e, n, m)
            tables.append(np.concatenate([h, np.ones_like(h)]))
        A = orc.m1_estimate(absnet, m, 0, 0, tables=tables, combine="dft", want_sketches=True)["sketches"]
        err = np.abs(got[r].cpu().numpy() - ref)
        assert np.all(err <= TAU["float64"] * A), (r, (err / A).max())

"""m above 16384: a slot's ranges of buckets on one block or shared by two or four, by how many blocks there are.  The
terms are summed in fixed point, so a sample's sketches are the same bit for bit whichever way it went, and they are
held against the FP64 oracle (bars as in test_gpu_scatter)."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import TAU, make_plan
from test_gpu_scatter import T  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m, dtype", [(65536, "float64"), (32768, "float64"), (65536, "float32")])
def test_ranges_shared(T, orc, m, dtype):  # noqa: F811
    rng = np.random.default_rng(5)
    shapes = [(600, 7), (7, 90), (90, 600)]  # two chunks of rows, rows of 7, of 90, of 600
    data = [rng.choice([-1.0, 1.0], s) * (0.5 + 0.5 * rng.random(s)) for s in shapes]
    net = W.Network([2, 2, 2], [n for s in shapes for n in s], [(1, 2), (3, 4), (5, 0)], data)
    S = 90  # 270 blocks, one per slot and sample
    plan, views = make_plan(T, [net], dtype, m, S, 40)
    whole = plan.sketches(first=0, count=S)
    for first, count in ((3, 1), (20, 36), (50, 40), (0, 21)):  # 3, 108, 120 and 63 blocks
        assert np.array_equal(plan.sketches(first=first, count=count).cpu().numpy(),
                              whole[first:first + count].cpu().numpy()), (first, count)
    absnet = views[0].with_data([np.abs(x) for x in views[0].data])
    for r in (0, S - 1):
        ref = orc.m1_estimate(views[0], m, 40, r, combine="dft", want_sketches=True)["sketches"]
        tables = []
        for e in range(net.t):
            h, _ = orc.hash_table(40, r, e, net.dims[net.edges[e][0]], m)
            tables.append(np.concatenate([h, np.ones_like(h)]))
        A = orc.m1_estimate(absnet, m, 0, 0, tables=tables, combine="dft", want_sketches=True)["sketches"]
        err = np.abs(whole[r].cpu().numpy() - ref)
        assert np.all(err <= TAU[dtype] * A + 1e-300), (r, (err - TAU[dtype] * A).max())

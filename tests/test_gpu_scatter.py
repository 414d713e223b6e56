"""The scatter's two kernels at the edges of their dispatch, sketches against the FP64 oracle bucket by bucket.

Slots of at most 1024 entries, of tensors of at most four modes of together at most 192 indices, take one wave per
sample (m <= 2048); all others a block whose hash words are staged under the same limits on the modes and read from
the global tables otherwise, 512 rows at a time; above m = 16384 it takes ranges of buckets in turn.  Entries have
magnitudes in [1/2, 1), so the fixed point's resolution (2^-46 of the largest entry per term) stays far below
tau * A_b (see test_gpu_m1)."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import TAU, make_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    import paper_2603_07387_amd as T
    assert torch.cuda.is_available()
    T.load()
    return T


def _ring(shapes, edges, seed):
    rng = np.random.default_rng(seed)
    data = [rng.choice([-1.0, 1.0], s) * (0.5 + 0.5 * rng.random(s)) for s in shapes]
    return W.Network([len(s) for s in shapes], [n for s in shapes for n in s], edges, data)


def networks():
    return [
        # 1020 rows of 3 (two chunks of rows, rows shorter than a vector), 192 and 194 words, five modes
        _ring([(1020, 3), (3, 189), (189, 5), (5, 2, 2, 3, 2), (2, 2, 3, 2, 1020)],
              [(1, 2), (3, 4), (5, 6), (7, 11), (8, 12), (9, 13), (10, 14), (15, 0)], 1),
        # 1024 entries, 800, 1025 and 1312
        _ring([(32, 32), (32, 25), (25, 41), (41, 32)], [(1, 2), (3, 4), (5, 6), (7, 0)], 2),
        # several slots of 1092 rows of 60 (staged words, three chunks each)
        _ring([(60, 60, 60), (60, 60, 60)], [(0, 5), (1, 4), (2, 3)], 3),
    ]


@pytest.mark.parametrize("m", [2, 512, 2048, 4096, 32768])
@pytest.mark.parametrize("dtype", ["float64", "float32", "bfloat16"])
def test_scatter_edges(T, orc, dtype, m):
    S = 9
    plan, views = make_plan(T, networks(), dtype, m, S, 40)
    got = plan.sketches(first=0, count=S).cpu().numpy()
    again = plan.sketches(first=4, count=5).cpu().numpy()
    assert np.array_equal(again, got[4:])  # exact integer sums: however the samples are grouped
    k0 = 0
    for j, net in enumerate(views):
        absnet = net.with_data([np.abs(x) for x in net.data])
        for r in (0, 5, S - 1):
            ref = orc.m1_estimate(net, m, 40 + j, r, combine="dft", want_sketches=True)["sketches"]
            tables = []
            for e in range(net.t):
                h, _ = orc.hash_table(40 + j, r, e, net.dims[net.edges[e][0]], m)
                tables.append(np.concatenate([h, np.ones_like(h)]))
            A = orc.m1_estimate(absnet, m, 0, 0, tables=tables, combine="dft", want_sketches=True)["sketches"]
            err = np.abs(got[r, k0:k0 + net.p] - ref)
            assert np.all(err <= TAU[dtype] * A + 1e-300), (j, r, (err - TAU[dtype] * A).max())
        k0 += net.p

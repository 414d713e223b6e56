"""The two-child gather at the edges of its range: second children of 1, 3, 255 and 256 values, first children beyond
a block's threads, sketch sizes from 2 to 8192 (one sample staged per block at the largest), sample counts that leave
a block one sample, leaf and non-leaf children in both places, against the FP64 oracle (bars as in test_gpu_m2)."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m2 import T, check, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


def _net(shapes, edges, seed):
    rng = np.random.default_rng(seed)
    return W.Network([len(s) for s in shapes], [n for s in shapes for n in s], edges,
                     [rng.standard_normal(s) / np.sqrt(s[-1]) for s in shapes])


def trains():
    # root (a, b), children: vector a, core (b, c, d) with a vector on c or on d, its other child a vector or core
    out = []
    for (b, c, d) in ((5, 300, 1), (7, 3, 255), (3, 2, 256), (70, 64, 3)):
        out.append(_net([(4, b), (4,), (b, c, d), (c,), (d,)], [(0, 2), (1, 3), (4, 6), (5, 7)], b))
        out.append(_net([(b, 4), (4,), (c, b, d), (c, 6), (6,), (d,)], [(1, 2), (0, 4), (3, 6), (7, 8), (5, 9)], c))
    return out


@pytest.mark.parametrize("m,S", [(2, 9), (64, 1), (1024, 11), (8192, 3)])
@pytest.mark.parametrize("dtype", ["float64", "float32", "bfloat16"])
def test_pair_edges(T, orc, dtype, m, S):  # noqa: F811
    plan, views = make_plan(T, trains(), dtype, m, S, 31)
    check(orc, plan, views, 31, dtype)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_all_pairs_many_samples(T, orc, dtype):  # noqa: F811
    """Every level two-child, staged several samples per block, partial sums of the level below."""
    net = W.tt_caterpillar(cores=4, bond=66, phys=33, seed=8, dtype=np.float64)
    plan, views = make_plan(T, [net], dtype, 512, 2600, 5)
    check(orc, plan, views, 5, dtype, samples=[0, 1, 2, 3, 1300, 2597, 2598, 2599])

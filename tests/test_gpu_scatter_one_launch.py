"""Slots of both kinds (a wave or a block to a sample) in one launch where they are few, in two otherwise: a sample's
sketches are the same bit for bit, so a call of few samples equals the same samples of a call of many."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import make_plan
from test_gpu_scatter import T  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 64, 2048])
@pytest.mark.parametrize("dtype", ["float64", "float32", "bfloat16"])
def test_one_and_two_launches(T, dtype, m):  # noqa: F811
    rng = np.random.default_rng(4)
    shapes = [(29,), (28, 8, 29), (300, 8), (32, 28), (32,), (300,), (1, 1), (1, 1), (1024,), (1024,)]
    dims = [n for s in shapes for n in s]
    edges = [(0, 3), (5, 2), (1, 7), (6, 8), (4, 9), (10, 12), (13, 11), (14, 15)]
    net = W.Network([len(s) for s in shapes], dims, edges, [rng.standard_normal(s) for s in shapes])
    S = 1700  # 10 slots of each of two networks: two launches for more than 409 samples (of four to a pass)
    plan, _ = make_plan(T, [net, net], dtype, m, S, 40)
    many = plan.sketches(first=0, count=S)
    for first, count in ((0, 3), (1000, 101), (1690, 10)):
        assert np.array_equal(plan.sketches(first=first, count=count).cpu().numpy(),
                              many[first:first + count].cpu().numpy()), (first, count)

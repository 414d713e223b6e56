"""The two-child gather with FP64 children of very different magnitudes: the fixed-point scale times one child's values
overflows where the other's are below 2^-972, though the products and the scale itself are ordinary numbers.  Against
the FP64 oracle (bars as in test_gpu_m2)."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m2 import T, check, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


def net(scale_c, scale_d, seed):
    # root (a, b) with the vector a and the core (b, c, d), whose children are the vectors c and d
    rng = np.random.default_rng(seed)
    shapes = [(6, 5), (6,), (5, 30, 7), (30,), (7,)]
    scales = [1.0, 1.0, 1.0, scale_c, scale_d]
    return W.Network([len(s) for s in shapes], [n for s in shapes for n in s], [(0, 2), (1, 3), (4, 6), (5, 7)],
                     [rng.standard_normal(s) * f for s, f in zip(shapes, scales)])


@pytest.mark.parametrize("scale_c, scale_d", [(1e-300, 1e150), (1e150, 1e-300), (1e-305, 1e170), (1e200, 1e90),
                                              (0.0, 1e200)])
def test_scales(T, orc, scale_c, scale_d):  # noqa: F811
    plan, views = make_plan(T, [net(scale_c, scale_d, k) for k in range(2)], "float64", 64, 5, 3)
    check(orc, plan, views, 3, "float64")

"""FP64 products over columns split into short ranges (two chunks at the least): column counts at and around the
splits' edges (a range that ends inside a chunk, one that is empty, no split at all), more rows than a tile, against
the FP64 oracle (bars as in test_gpu_m2)."""
import pytest

import tn_workloads as W
import numpy as np
from test_gpu_m2 import T, check, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bond,phys", [(3, 20), (8, 16), (43, 3), (17, 15), (16, 16), (27, 20), (70, 15)])
@pytest.mark.parametrize("dtype", ["float64", "float32", "bfloat16"])
def test_split_edges(T, orc, dtype, bond, phys):  # noqa: F811
    net = W.tt_caterpillar(cores=4, bond=bond, phys=phys, seed=bond, dtype=np.float64)
    plan, views = make_plan(T, [net], dtype, 256, 65, 7)
    check(orc, plan, views, 7, dtype, samples=[0, 1, 63, 64])

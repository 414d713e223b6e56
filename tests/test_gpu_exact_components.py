"""tn_contract_exact on networks of several components: the run lays its tensors out in the arena exactly as the dry
run did, also from the second component on (whose first free place depends on the first one's result being given back).
Values against FP64 einsum; bars as in test_gpu_exact_trees."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_exact import einsum_value, exact

pytestmark = pytest.mark.gpu


def from_labels(tensors, sizes, seed):
    flat = [e for t in tensors for e in t]
    edges = [tuple(u for u, x in enumerate(flat) if x == e) for e in range(len(sizes))]
    rng = np.random.default_rng(seed)
    return W.Network([len(t) for t in tensors], [sizes[e] for e in flat], edges,
                     [rng.standard_normal([sizes[e] for e in t]) for t in tensors])


SIX = [[0], [0], [1, 2, 4, 5, 6], [1], [2, 3, 6], [3, 4, 5]]
CASES = {
    "two components": (SIX, [6, 4, 2, 3, 2, 6, 3]),
    "three": (SIX + [[7, 8], [8, 7]], [6, 4, 2, 3, 2, 6, 3, 40, 7]),
    "the large one first": ([[1, 2, 4, 5, 6], [1], [2, 3, 6], [3, 4, 5], [0], [0]], [6, 4, 2, 3, 2, 6, 3]),
    "scalars of traces": ([[0, 0], [1, 1], [2], [2]], [300, 5, 70]),
}


@pytest.mark.parametrize("case", list(CASES))
def test_components(case):
    import paper_2603_07387_amd as T
    net = from_labels(*CASES[case], seed=len(case))
    got, view = exact(T, net, "float64")
    want = einsum_value(view)
    scale = einsum_value(view.with_data([np.abs(x) for x in view.data]))
    assert abs(got - want) <= 1e-12 * scale

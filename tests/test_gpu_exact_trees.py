"""tn_contract_exact over random networks (traces, several components, labels
of dimension 1, up to 16 tensors for the subset search and more for the greedy
tree) against FP64 einsum.  Every product and sum is FP64 on both sides, in
another order: an entry of a result of up to 2^14 terms and 20 steps is off by
well under 1e-12 times the contraction of the absolute values."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_exact import einsum_value, exact

pytestmark = pytest.mark.gpu


def network(p, seed):
    rng = np.random.default_rng(seed)
    ends, dims = [], []
    for k in range(1, p):
        if rng.random() < 0.9:
            ends.append((k, int(rng.integers(0, k))))  # else: a component of its own
    ends += [(int(rng.integers(0, p)), int(rng.integers(0, p))) for _ in range(p // 2)]  # traces among them
    ends += [(k, k) for k in range(p) if not any(k in e for e in ends)]
    dims = [int(rng.integers(1, 5)) for _ in ends]
    modes = [[] for _ in range(p)]
    for e, (a, b) in enumerate(ends):
        modes[a].append(e)
        modes[b].append(e)
    orders = [len(x) for x in modes]
    flat = [e for x in modes for e in x]
    edges = [tuple(u for u, e2 in enumerate(flat) if e2 == e) for e in range(len(ends))]
    data, u = [], 0
    for q in orders:
        data.append(rng.standard_normal([dims[e] for e in flat[u:u + q]]))
        u += q
    return W.Network(orders, [dims[e] for e in flat], edges, data)


@pytest.mark.parametrize("p", [1, 2, 3, 7, 12, 16, 18])
@pytest.mark.parametrize("seed", range(3))
def test_random_networks(p, seed):
    import paper_2603_07387_amd as T
    net = network(p, 10 * p + seed)
    got, view = exact(T, net, "float64")
    want = einsum_value(view)
    scale = einsum_value(view.with_data([np.abs(x) for x in view.data]))
    assert abs(got - want) <= 1e-12 * scale

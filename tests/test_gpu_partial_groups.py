"""Partial contraction with its tensor pairs in two groups: every entry against
the FP64 combine of the plan's own sketches, (1/m) sum_j prod_k FFT(y_k)[j].

The pair transforms run in the data's accumulation type A (unit roundoff u):
an FFT of m points is off by at most about 3 log2(m) u times its input's
2-norm in norm, so each of p factors is off by that relative to sqrt(m)
||y_k||, and an entry by p times it, times prod_k ||y_k|| sqrt(m)^(p - 2) / 1
(Cauchy-Schwarz over two factors, the others bounded by sqrt(m) ||y||): with
two tensors to a transform, twice.  Networks: free modes in one group only,
in both, an odd tensor out, sizes off the 16 x 16 tiles, every short m."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import dev

pytestmark = pytest.mark.gpu


def ring(p, contracted, free):
    """p tensors in a ring of contractions; tensor k with free modes free[k] of which the first leads."""
    orders, dims, edges, u = [], [], [], 0
    left, right = [], []
    for k in range(p):
        f = free.get(k, [])
        lead, trail = f[:1], f[1:]
        orders.append(len(f) + 2)
        dims += lead + [contracted, contracted] + trail
        left.append(u + len(lead))
        right.append(u + len(lead) + 1)
        u += len(f) + 2
    for k in range(p):
        edges.append((right[k], left[(k + 1) % p]))
    rng = np.random.default_rng(p * 100 + len(free))
    data, u = [], 0
    for q in orders:
        data.append(rng.standard_normal(dims[u:u + q]))
        u += q
    return W.Network(orders, dims, edges, data)


CASES = [
    (5, {0: [17], 2: [3]}, 256, "float32"),          # 17 + 3 assignments, an odd tensor out
    (6, {0: [4, 5], 1: [3], 3: [2, 2]}, 64, "float64"),  # 60 x 4, trailing free modes
    (8, {2: [33]}, 1024, "float32"),                 # one group with free modes, the other with none
    (7, {0: [6], 3: [5], 4: [4], 6: [3]}, 2048, "bfloat16"),  # several pairs to a group
    (5, {0: [16], 2: [16]}, 2, "float64"),
    (5, {0: [9], 3: [9]}, 1, "float32"),
    (5, {1: [5], 2: [4]}, 8192, "float64"),
]


@pytest.mark.parametrize("p, free, m, dtype", CASES)
def test_entries(p, free, m, dtype):
    import torch
    import paper_2603_07387_amd as T
    net = ring(p, 5, free)
    S = 2048 // int(np.prod([n for f in free.values() for n in f])) + 1  # entries x samples of the grouped way
    ts = dev(net, dtype)
    plan = T.PartialPlan(T.NetworkSpec.from_network(net, ts), m, S, 11)
    got = torch.empty(plan.n_nets * S, dtype=torch.float64, device="cuda")
    plan.estimate(samples_out=got)
    y = plan.sketches(0, S)
    torch.cuda.synchronize()
    got = got.cpu().numpy().reshape(*plan.out_shape, S)
    y = y.cpu().numpy().reshape(S, -1, m)
    spec = np.fft.fft(y, axis=2)
    norm = np.linalg.norm(y, axis=2)
    first, size = [], []
    for k in range(p):
        first.append(sum(size))
        size.append(int(np.prod(free.get(k, [1]))))
    u = 2.0 ** (-53 if dtype == "float64" else -24)
    checked = 0
    for r in np.ndindex(*plan.out_shape):
        digits = list(r)
        prod, bound = 1.0, 1.0
        for k in range(p):
            v = 0
            for n in free.get(k, []):
                v = v * n + digits.pop(0)
            prod = prod * spec[:, first[k] + v]
            bound = bound * norm[:, first[k] + v]
        want = prod.real.mean(axis=1)
        tol = 2 * p * (3 * max(1, np.log2(m)) + 4) * u * bound * np.sqrt(m) ** (p - 2)
        assert np.all(np.abs(got[r] - want) <= tol), (r, np.abs(got[r] - want) / tol)
        checked += 1
    assert checked == plan.n_nets

"""m >= 2^15 with FP32 sketches: the scatter that takes the combine's first
transforms with it, against the plan that keeps its sketches (TN_FLAG_RESIDENT:
scatter, then transforms).  Both add the same terms in 64-bit fixed point and
take the same FP32 transforms, so the estimates are equal bit for bit.

Cases: columns fewer than four and up to 1024, more rows than columns and the
reverse, one-mode tensors, an odd tensor out, few blocks (a pair's ranges on
several blocks) and many, several chunks of samples, and a plan with a tensor
of two slots, which goes the other way."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import dev

pytestmark = pytest.mark.gpu


def ring(*bonds):
    """Matrices in a cycle: bonds[k] x bonds[k + 1]."""
    p = len(bonds)
    dims = [d for k in range(p) for d in (bonds[k], bonds[(k + 1) % p])]
    return network([2] * p, dims, [(2 * k + 1, (2 * k + 2) % (2 * p)) for k in range(p)])


def network(orders, dims, edges):
    rng = np.random.default_rng(len(dims))
    data, u = [], 0
    for q in orders:
        data.append(rng.standard_normal(dims[u:u + q]))
        u += q
    return W.Network(orders, dims, edges, data)


CASES = {
    "torus": ([W.torus(L=3, D=8, seed=6, dist="normal")], 65536, 5, "float32"),
    "torus, bf16": ([W.torus(L=4, D=7, seed=6, dist="uniform")] * 3, 32768, 3, "bfloat16"),
    "thin": ([ring(3, 300, 2, 1024, 1)], 65536, 4, "float32"),
    "long rows": ([ring(513, 900, 64)], 32768, 7, "float32"),
    "vectors": ([network([1, 2, 1], [70, 70, 31, 31], [(0, 1), (2, 3)])] * 9, 32768, 6, "bfloat16"),
    "many": ([ring(40, 33, 50)] * 150, 65536, 4, "float32"),
    "two slots": ([ring(300, 300, 20)], 65536, 3, "float32"),
    "beyond the LDS": ([ring(60, 1024, 1024, 60)], 32768, 2, "float32"),
}


@pytest.mark.parametrize("case", list(CASES))
def test_equals_the_kept_sketches(case):
    import torch
    import paper_2603_07387_amd as T
    nets, m, S, dtype = CASES[case]
    specs, hold = [], []
    for k, net in enumerate(nets):
        ts = dev(net.with_data([x * (1.0 + k) for x in net.data]), dtype)
        hold.append(ts)
        specs.append(T.NetworkSpec.from_network(net, ts))
    got = []
    for flags in (0, T.TN_FLAG_RESIDENT):
        plan = T.Plan(specs, T.TN_CYCLIC, m, S, 3, flags=flags)
        out = torch.empty(len(nets) * S, dtype=torch.float64, device="cuda")
        plan.estimate(samples_out=out)
        plan.estimate(samples_out=out)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
        plan.close()
    assert np.any(got[0] != 0.0)
    assert np.array_equal(got[0], got[1])

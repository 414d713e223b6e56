"""Scatter blocks of 256 threads (every slot small, many blocks) and column words formed once per block, against the
same networks in plans of their own (512 threads): the terms are summed in fixed point, so the estimates are equal bit
for bit.  Edges: rows plus columns of 512 and one more, ragged columns, slots of the largest size that counts."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a, b, c, m, dtype", [
    (64, 64, 64, 256, "float64"), (256, 256, 4, 64, "float32"), (257, 256, 3, 64, "float32"),
    (37, 51, 90, 1024, "bfloat16"), (16384, 1, 2, 256, "float32"), (128, 128, 127, 2048, "float64")])
def test_equals_single_networks(a, b, c, m, dtype):
    import torch
    import paper_2603_07387_amd as T
    count, S = 40, 77
    rng = np.random.default_rng(a + b)
    specs, hold = [], []
    for _ in range(count):
        first = (a,) if a <= 1024 else (a // 1024, 1024)
        orders = [len(first) + 1, 2, 1 + len(first)]
        dims = list(first) + [b, b, c, c] + list(first)
        u = [0] + list(np.cumsum(orders))
        edges = [(u[1] - 1, u[1]), (u[2] - 1, u[2])] + [(i, u[2] + 1 + i) for i in range(len(first))]
        data, at = [], 0
        for q in orders:
            data.append(rng.standard_normal(dims[at:at + q]))
            at += q
        net = W.Network(orders, dims, edges, data)
        ts = dev(net, dtype)
        hold.append(ts)
        specs.append(T.NetworkSpec.from_network(net, ts))

    def run(sp, seed):
        plan = T.Plan(sp, T.TN_CYCLIC, m, S, seed)
        out = torch.empty(len(sp) * S, dtype=torch.float64, device="cuda")
        plan.estimate(samples_out=out)
        torch.cuda.synchronize()
        return out.cpu().numpy().reshape(len(sp), S)

    got = run(specs, 5)
    for j in (0, 1, 17, count - 1):
        assert np.array_equal(got[j], run([specs[j]], 5 + j)[0]), j

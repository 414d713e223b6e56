"""Hash tables of streams of more than 64 indices at the edges of the lane rule (64 indices to a lane, all 64 lanes
above 512), few and many pairs, against the oracle's family."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S, dims", [(3, (512, 513, 1)), (6000, (65, 128, 129)), (5500, (300, 512, 7)),
                                     (5500, (513, 3, 64)), (1400, (1024, 2, 1023)), (700, (3000, 2, 1))])
def test_long_streams(orc, S, dims):
    import paper_2603_07387_amd as T
    a, b, c = dims
    if a <= 1024:
        net = W.Network([2, 2, 2], [a, b, b, c, c, a], [(1, 2), (3, 4), (5, 0)],
                        [np.ones((a, b)), np.ones((b, c)), np.ones((c, a))])
    else:  # a long first mode
        net = W.Network([2, 3, 1], [a, b, a, b, c, c], [(0, 2), (1, 3), (4, 5)],
                        [np.ones((a, b)), np.ones((a, b, c)), np.ones(c)])
    plan = T.Plan([T.NetworkSpec.from_network(net, dev(net, "float32"))], T.TN_CYCLIC, 64, S, 9)
    got = plan.hashes().cpu().numpy()
    for s in sorted({0, S // 2, S - 1}):
        for (_, sid, n, off) in plan.streams():
            h, sg = orc.hash_table(9, s, sid, n, 64)
            v = got[s, off:off + n]
            assert np.array_equal(v & 0x7FFFFFFF, h), (s, sid)
            assert np.array_equal(np.where(v < 0, -1, 1), sg), (s, sid)


def test_more_threads_than_a_grid_row(orc):
    """One stream of 600 indices among 3003, 24000 samples: 64 lanes to each of 72 million pairs is more than 2^32
    threads."""
    import torch
    import paper_2603_07387_amd as T
    x, one = torch.ones(600, 1, device="cuda"), torch.ones(1, 1, device="cuda")
    edges = [(1, 2), (3, 4), (5, 0)]
    specs = [T.NetworkSpec([2, 2, 2], [600, 1, 1, 1, 1, 600], edges, tensors=[x, one, x.view(1, 600)])]
    specs += [T.NetworkSpec([2, 2, 2], [1] * 6, edges, tensors=[one] * 3)] * 1000
    plan = T.Plan(specs, T.TN_CYCLIC, 64, 24000, 9)
    got = plan.hashes()
    streams = plan.streams()
    for k in (0, 1, 2, 1500, 3002):
        net, sid, n, off = streams[k]
        for s in (0, 11999, 23999):
            h, sg = orc.hash_table(9 + net, s, sid, n, 64)
            v = got[s, off:off + n].cpu().numpy()
            assert np.array_equal(v & 0x7FFFFFFF, h), (k, s)
            assert np.array_equal(np.where(v < 0, -1, 1), sg), (k, s)

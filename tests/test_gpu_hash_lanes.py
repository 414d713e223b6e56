"""Hash tables with one to 64 lanes per (stream, sample): pair counts around
the rule's edges, streams of 1 to 65 indices, against the oracle's family."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S, dims", [(1, (1, 65, 2)), (16, (64, 64, 64)), (1365, (3, 7, 33)), (1366, (3, 7, 33)),
                                     (21846, (2, 5, 4)), (65535, (1, 1, 3))])
def test_hash_tables(orc, S, dims):
    import torch
    import paper_2603_07387_amd as T
    a, b, c = dims
    net = W.Network([2, 2, 2], [a, b, b, c, c, a], [(1, 2), (3, 4), (5, 0)],
                    [np.ones((a, b)), np.ones((b, c)), np.ones((c, a))])
    plan = T.Plan([T.NetworkSpec.from_network(net, dev(net, "float32"))], T.TN_CYCLIC, 64, S, 9)
    got = plan.hashes().cpu().numpy()
    for s in sorted({0, 1 % S, S // 2, S - 1}):
        for (_, sid, n, off) in plan.streams():
            h, sg = orc.hash_table(9, s, sid, n, 64)
            v = got[s, off:off + n]
            assert np.array_equal(v & 0x7FFFFFFF, h), (s, sid)
            assert np.array_equal(np.where(v < 0, -1, 1), sg), (s, sid)

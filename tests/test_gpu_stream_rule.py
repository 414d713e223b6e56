"""Turnstile updates on both sides of the rule that sums them in shares (n >= m and n S >= 16 m): one call against
the same updates in two calls of half, which go the other way or are shared otherwise.  Whole numbers sum exactly, so
the estimates are equal bit for bit."""
import numpy as np
import pytest

from test_gpu_m1 import dev
from test_gpu_stream_shares import triangle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m, S, n, dtype", [
    (16384, 15, 16384, "float32"), (16384, 16, 16384, "float32"), (16384, 1, 262144, "float64"),
    (4096, 3, 16384, "float64"), (4096, 4, 16384, "float64"), (64, 16, 64, "float32"), (64, 17, 63, "float32"),
    (1, 16, 2, "float32"), (32768, 2, 524288, "float32")])
def test_rule(m, S, n, dtype):
    import torch
    import paper_2603_07387_amd as T
    net = triangle(37, 50, 3, extra=5)
    spec = T.NetworkSpec.from_network(net, dev(net, dtype))
    rng = np.random.default_rng(m + n)
    feeds = []
    for k in range(3):
        idx = rng.integers(-3, int(np.prod(net.shape(k))) + 3, n)  # some outside the tensor: ignored
        feeds.append((torch.from_numpy(idx).cuda(), torch.from_numpy(rng.integers(-4, 5, n).astype(np.float64)).cuda()))
    got = []
    for step in (n, (n + 1) // 2):
        plan = T.Plan([spec], T.TN_CYCLIC, m, S, 5, flags=T.TN_FLAG_RESIDENT)
        plan.reset()
        for k, (i, d) in enumerate(feeds):
            for u in range(0, n, step):
                plan.update(k, i[u:u + step].clone(), d[u:u + step].clone())
        out = torch.empty(S, dtype=torch.float64, device="cuda")
        plan.combine(samples_out=out)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
        plan.close()
    assert np.array_equal(got[0], got[1])
    assert np.any(got[0] != 0.0)

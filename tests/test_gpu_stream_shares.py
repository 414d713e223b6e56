"""Turnstile updates by shares (at least m of them in a call: summed per block
in LDS, then added to the sketch) against the same updates fed a few at a time,
and the combine's wide blocks and slot loads against the FP64 combine of the
plan's sketches.

Whole-number updates sum exactly in FP32 and FP64 in any order, so the two
routes leave the same sketches and the estimates are equal bit for bit."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_m1 import dev

pytestmark = pytest.mark.gpu


def triangle(n0, n1, n2, extra=1):
    """Three matrices in a cycle; the first with a third mode of size `extra` that the second shares."""
    orders, dims = [3, 3, 2], [n0, extra, n1, n1, extra, n2, n2, n0]
    return W.Network(orders, dims, [(2, 3), (1, 4), (5, 6), (7, 0)],
                     [np.zeros((n0, extra, n1)), np.zeros((n1, extra, n2)), np.zeros((n2, n0))])


@pytest.mark.parametrize("m, S, n, dtype", [
    (64, 300, 64, "float32"), (64, 7, 63, "float64"), (1, 3, 5, "float32"), (256, 1, 70001, "float64"),
    (4096, 5, 4099, "float32"), (4096, 5, 8191, "float64"), (16384, 3, 40000, "float32"), (32768, 2, 40000, "float32"),
    (1024, 60000, 1030, "float32")])
def test_shares_equal_single_updates(m, S, n, dtype):
    import torch
    import paper_2603_07387_amd as T
    net = triangle(37, 50, 3, extra=5)
    ts = dev(net, dtype)
    spec = T.NetworkSpec.from_network(net, ts)
    rng = np.random.default_rng(m + n)
    feeds = []
    for k in range(3):
        size = int(np.prod(net.shape(k)))
        idx = rng.integers(-3, size + 3, n)  # some outside the tensor: ignored
        feeds.append((torch.from_numpy(idx).cuda(), torch.from_numpy(rng.integers(-4, 5, n).astype(np.float64)).cuda()))
    got = []
    few = max(1, min(m - 1, 2000))
    for step in (n, few):  # m = 1: no call of fewer updates than m, the routes are the same
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


@pytest.mark.parametrize("m, S, dtype", [(4096, 3, "float32"), (2048, 150, "float32"), (4096, 90, "float64"),
                                         (1024, 5, "float64"), (8192, 2, "float32")])
def test_combine_of_many_slots(m, S, dtype):
    """Tensors of 1 to 6 slots, blocks above and below one to a CU.  Per sample the combine's FP error: three
    factors, each off by at most 4 log2(m) + 8 roundings of its norm (its slots' sums and the transform), twice
    for the two tensors of a transform, times the product of the norms, sqrt(m) for the factor left over."""
    import torch
    import paper_2603_07387_amd as T
    net = triangle(1000, 1000, 7, extra=5)
    rng = np.random.default_rng(3)
    net = W.Network(net.orders, net.dims, net.edges, [rng.standard_normal(net.shape(k)) for k in range(3)])
    ts = dev(net, dtype)
    plan = T.Plan([T.NetworkSpec.from_network(net, ts)], T.TN_CYCLIC, m, S, 5)
    out = torch.empty(S, dtype=torch.float64, device="cuda")
    plan.estimate(samples_out=out)
    y = plan.sketches(0, S)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    want = np.fft.fft(y, axis=2).prod(axis=1).real.mean(axis=1)
    u = 2.0 ** (-53 if dtype == "float64" else -24)
    tol = 2 * 3 * (4 * np.log2(m) + 8) * u * np.linalg.norm(y, axis=2).prod(axis=1) * np.sqrt(m)
    assert np.all(np.abs(out.cpu().numpy() - want) <= tol)

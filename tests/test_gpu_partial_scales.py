"""Grouped partial contraction of FP64 tensors whose pairs are far apart in magnitude: the product over one group alone
leaves the range of FP64 (2^1320, and 2^-1320 in the other), the whole product does not.  Every tensor is an ordinary
one times a power of two, so each sample is that of the ordinary network, bit for bit, times the powers' product (the
two tensors of a transform by the same power: they share its rounding)."""
import numpy as np
import pytest

from test_gpu_m1 import dev
from test_gpu_partial_groups import ring

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, powers, dtype", [
    (5, [330, 330, -330, -330, 330, 330, -330, -330], "float64"),   # one wave per sample
    (5, [0, 0, 3, 3, -5, -5, 2, 2], "float64"),
    (40, [330, 330, -330, -330, 330, 330, -330, -330], "float64"),  # blocks
    (5, [60, 60, -60, -60, 60, 60, -60, -60], "float32")])
def test_scaled_pairs(n, powers, dtype):
    import torch
    import paper_2603_07387_amd as T
    net = ring(8, n, {0: [30], 2: [40], 4: [2]})  # pairs 1 and 3 to one group, 0 and 2 to the other
    got = []
    for pw in ([0] * 8, powers):
        scaled = net.with_data([np.ldexp(x.astype(np.float32).astype(np.float64), e) for x, e in zip(net.data, pw)])
        ts = dev(scaled, dtype)
        plan = T.PartialPlan(T.NetworkSpec.from_network(scaled, ts), 256, 3, 11)
        out = torch.empty(plan.n_nets * 3, dtype=torch.float64, device="cuda")
        plan.estimate(samples_out=out)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    assert np.all(np.isfinite(got[0])) and np.any(got[0] != 0.0)
    assert sum(powers) == 0
    assert np.array_equal(got[0], got[1])


def test_many_fp32_pairs():
    """Twenty FP32 tensors, seven pairs in one group, five of them large: 2^1040 there.  The small tensors' transforms
    come within 2^-45 of their norm of the smallest numbers of FP32, so samples agree to far better than 2^-30 of the
    largest only."""
    import torch
    import paper_2603_07387_amd as T
    net = ring(20, 3, {2 * j: [f] for j, f in enumerate((4, 3, 3, 3, 2, 2, 1, 1, 1, 1))})  # groups 0 3 5 and the others
    net = net.with_data([x.astype(np.float32).astype(np.float64) for x in net.data])
    large = np.repeat([104 if j in (1, 2, 4, 6, 7) else -104 for j in range(10)], 2)
    got = []
    for powers in ([0] * 20, large):
        scaled = net.with_data([np.ldexp(x, int(e)) for x, e in zip(net.data, powers)])
        ts = dev(scaled, "float32")
        plan = T.PartialPlan(T.NetworkSpec.from_network(scaled, ts), 64, 5, 11)
        out = torch.empty(plan.n_nets * 5, dtype=torch.float64, device="cuda")
        plan.estimate(samples_out=out)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    assert np.all(np.isfinite(got[0])) and np.any(got[0] != 0.0)
    assert np.all(np.abs(got[0] - got[1]) <= 2.0 ** -30 * np.abs(got[0]).max())

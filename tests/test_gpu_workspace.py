"""Plans whose samples take more than one pass of the workspace, and what a plan asks of it.

Sketches are sums in fixed point and every sample is transformed by itself, so a plan's samples are the same bit for
bit however they are cut into passes (the later ones start from the largest entries that the first recorded)."""
import numpy as np
import pytest

import tn_workloads as W
from test_gpu_big_scatter import ring
from test_gpu_m1 import dev
from test_gpu_partial_groups import ring as partial_ring

pytestmark = pytest.mark.gpu


def make(T, nets, m, S, dtype, flags=0, scale=1.0):
    specs, hold = [], []
    for k, net in enumerate(nets):
        ts = dev(net.with_data([x * (scale + k) for x in net.data]), dtype)
        hold.append(ts)
        specs.append(T.NetworkSpec.from_network(net, ts))
    return T.Plan(specs, T.TN_CYCLIC, m, S, 3, flags=flags), hold


def samples(plan):
    import torch
    out = torch.empty(plan.n_nets * plan.S, dtype=torch.float64, device="cuda")
    plan.estimate(samples_out=out)
    plan.estimate(samples_out=out)
    torch.cuda.synchronize()
    return out.cpu().numpy().reshape(plan.n_nets, plan.S)


CASES = {
    # m >= 2^15, FP32: scatter and first transforms in one kernel; FP64: ranges of buckets
    "lattice, m = 65536": ([W.torus(L=3, D=8, seed=6, dist="normal")], 65536, 40, "float32", 64),
    "ragged, m = 32768, bf16": ([ring(40, 33, 50), ring(3, 300, 2, 1024, 1)], 32768, 9, "bfloat16", 8),
    "lattice, m = 32768, FP64": ([W.torus(L=3, D=6, seed=6, dist="normal")], 32768, 9, "float64", 16),
    # slots of several sizes, both kernels
    "m = 1024": ([ring(64, 20, 30), ring(100, 130, 300), ring(7, 5, 6)], 1024, 77, "float32", 1),
    "m = 256, FP64": ([ring(64, 20, 30), ring(100, 130, 300), ring(7, 5, 6)], 256, 24, "float64", 1),
}


@pytest.mark.parametrize("case", list(CASES))
def test_passes(case, monkeypatch):
    import paper_2603_07387_amd as T
    nets, m, S, dtype, mb = CASES[case]
    whole, hold = make(T, nets, m, S, dtype, flags=T.TN_FLAG_RESIDENT)
    want = samples(whole)
    monkeypatch.setenv("TN_WORKSPACE_MB", str(mb))
    plan, hold2 = make(T, nets, m, S, dtype)
    assert plan.query(9) < S  # several passes
    got = samples(plan)
    assert np.any(got != 0.0)
    assert np.array_equal(got, want)
    assert np.array_equal(plan.sketches(0, S).cpu().numpy(), whole.sketches(0, S).cpu().numpy())


def test_unused_sketches_take_no_room(monkeypatch):
    """9 tensors, m = 65536: 2.4 MB of sketches and 2.6 MB of transforms per sample; estimates keep the latter only.
    Exported sketches come in several pieces."""
    import paper_2603_07387_amd as T
    net = W.torus(L=3, D=8, seed=6, dist="normal")
    monkeypatch.setenv("TN_WORKSPACE_MB", "64")
    plan, _ = make(T, [net], 65536, 30, "float32")
    assert plan.query(9) >= 16
    monkeypatch.delenv("TN_WORKSPACE_MB")
    plan, _ = make(T, [net], 65536, 130, "float32")
    whole, _ = make(T, [net], 65536, 130, "float32", flags=T.TN_FLAG_RESIDENT)
    for first, count in ((0, 130), (100, 30), (129, 1)):
        assert np.array_equal(plan.sketches(first, count).cpu().numpy(), whole.sketches(first, count).cpu().numpy())


def test_smaller_workspace_after_out_of_memory(monkeypatch):
    """A workspace that the device does not have (537 GB of sketches): the plan takes one of 1 GiB instead."""
    import paper_2603_07387_amd as T
    net = ring(*[4] * 16)
    few, _ = make(T, [net], 65536, 16, "float64")
    monkeypatch.setenv("TN_WORKSPACE_MB", "4000000")
    plan, _ = make(T, [net], 65536, 65535, "float64")
    assert 1 <= plan.query(9) * 16 * 65536 * 8 <= 1 << 30
    assert np.array_equal(plan.sketches(0, 16).cpu().numpy(), few.sketches(0, 16).cpu().numpy())
    plan.close()


def test_partial_spectra_in_parts():
    """Grouped partial contraction whose spectra (2016 assignments, 16.5 MB per sample) pass their limit: the samples
    go in parts.  Entries against the FP64 combine of the plan's sketches; bars as in test_gpu_partial_groups."""
    import torch
    import paper_2603_07387_amd as T
    p, m, S = 4, 1024, 20
    free = {0: [50, 40], 2: [16]}
    net = partial_ring(p, 5, free)
    ts = dev(net, "float32")
    plan = T.PartialPlan(T.NetworkSpec.from_network(net, ts), m, S, 11)
    got = torch.empty(plan.n_nets * S, dtype=torch.float64, device="cuda")
    plan.estimate(samples_out=got)
    y = plan.sketches(0, S)
    torch.cuda.synchronize()
    got = got.cpu().numpy().reshape(2000, 16, S)
    y = y.cpu().numpy().reshape(S, -1, m)
    assert y.shape[1] == 2000 + 1 + 16 + 1
    spec = np.fft.rfft(y, axis=2)
    norm = np.linalg.norm(y, axis=2)
    wt = np.full(m // 2 + 1, 2.0)
    wt[[0, -1]] = 1.0
    u = 2.0 ** -24
    rng = np.random.default_rng(1)
    for a, b in zip(rng.integers(0, 2000, 300), rng.integers(0, 16, 300)):
        k = [a, 2000, 2001 + b, 2017]
        want = (np.prod([spec[:, i] for i in k], axis=0).real * wt).sum(axis=1) / m
        bound = np.prod([norm[:, i] for i in k], axis=0)
        tol = 2 * p * (3 * np.log2(m) + 4) * u * bound * np.sqrt(m) ** (p - 2)
        assert np.all(np.abs(got[a, b] - want) <= tol), (a, b)


def test_every_sample_the_same_for_every_schedule(monkeypatch):
    """Samples per pass, banks and the autotuner's choice change no bit of any sample, the first ones included."""
    import paper_2603_07387_amd as T
    rng = np.random.default_rng(17)
    big = rng.standard_normal((64, 128))
    big[-1, -1] = 8.0 * np.abs(big).max()  # the largest entry at the end
    late = W.Network([2, 2], [64, 128, 128, 64], [(0, 3), (1, 2)], [big, rng.standard_normal((128, 64))])
    nets = [W.torus(L=2, D=16, seed=9), W.random_network(4, 3), late]
    want = None
    for banks in ("1", "2"):
        for sb in ("1", "2", "4", "8"):
            monkeypatch.setenv("TN_SCATTER_BANKS", banks)
            monkeypatch.setenv("TN_SCATTER_SB", sb)
            plan, _ = make(T, nets, 1024, 24, "float32")
            assert plan.query(8) == int(sb) and plan.query(10) == int(banks)
            got = samples(plan)
            want = got if want is None else want
            assert np.array_equal(got, want), (banks, sb)
    monkeypatch.delenv("TN_SCATTER_BANKS")
    monkeypatch.delenv("TN_SCATTER_SB")
    plan, _ = make(T, nets, 1024, 24, "float32", flags=T.TN_FLAG_AUTOTUNE)
    got = samples(plan)
    assert plan.query(8) in (1, 2, 4, 8)
    assert np.array_equal(got, want)

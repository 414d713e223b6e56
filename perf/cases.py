"""The estimators' workloads, each a call that a user's program makes, for timing and for comparison in 64 bits.

listed() names the fixed cases, draw(rng) gives more of the same ranges.  A case is a dict of plain values;
prepare(case, seed) builds what the program holds before the call (device tensors made from the seed, the plan),
run(state) makes the call and returns its outputs, work(case) states the bytes and operations the call cannot do
without, and exact(case, seed) computes the same outputs in 64 bits with plain torch and numpy.

Kinds:
  triangle   tr(ABC) of n x n matrices, `count` networks in one plan (cyclic method)
  batch      `count` random connected cyclic networks of 3 to 12 tensors, bonds 2 to 32 (cyclic method)
  torus      side x side periodic lattices of order-4 tensors, U[0, 1) (cyclic method)
  ladder     the inner product of two tensor trains (cyclic method)
  tree       a tensor train whose physical legs meet vectors (acyclic method)
  partial    every entry of the output of a 3 x 3 torus with two contractions cut (partial contraction)
  stream     a directed edge stream into resident triangle sketches, then their estimates (turnstile updates)
  exact      the exact FP64 contraction of a torus, the reference value
  train      one epoch of the sketch-size regressor's training
"""
from __future__ import annotations

import functools
import math
import random

import numpy as np
import torch

import paper_2603_07387_amd as T

DTYPES = {"float64": torch.float64, "float32": torch.float32, "bfloat16": torch.bfloat16}
ESIZE = {"float64": 8, "float32": 4, "bfloat16": 2}
P31 = 2147483647


def listed():
    return [
        # one small network, one plan: the unbatched call, where launches and host work are most of the time
        dict(name="triangle_one", kind="triangle", count=1, n=64, m=256, samples=16, dtype="float64", graph=False),
        # the benchmark's batch: thousands of small networks of ragged shapes, matrix-core combine, tuned schedule
        dict(name="batch_4096", kind="batch", count=4096, m=1024, samples=16, dtype="float32", dft="bf16", tune=True),
        # a smaller batch of 16-bit data, FFT combine, untuned: a program that plans a new batch for each call
        dict(name="batch_bf16", kind="batch", count=200, m=512, samples=24, dtype="bfloat16", dft="fft", tune=False),
        # the benchmark's lattices: large equal tensors, many passes over them
        dict(name="torus_256", kind="torus", count=256, side=4, bond=16, m=1024, samples=32, dtype="float32", tune=True),
        # the largest sketch: its buckets and its transform do not fit on chip
        dict(name="torus_m65536", kind="torus", count=48, side=4, bond=16, m=65536, samples=6, dtype="float32",
             tune=False),
        # one network of many tensors, a long product
        dict(name="ladder", kind="ladder", count=1, cores=32, bond=64, phys=64, m=4096, samples=64, dtype="float32",
             tune=True),
        # the benchmark's tree: a deep chain of products over thousands of samples, FP32 matrix cores
        dict(name="caterpillar", kind="tree", count=1, cores=32, bond=64, phys=64, m=4096, samples=4096,
             dtype="float32", products="f32"),
        # FP64 trees of odd sizes, several in one plan: the acyclic method's reference mode
        dict(name="trees_f64", kind="tree", count=6, cores=9, bond=27, phys=20, m=1024, samples=500, dtype="float64",
             products="f64"),
        # partial contraction: 4096 output entries from shared sketches
        dict(name="partial", kind="partial", bond=8, m=1024, samples=8, dtype="float32"),
        # triangle counting over an edge stream with deletions
        dict(name="stream", kind="stream", vertices=1024, edges=32768, m=4096, samples=32, dtype="float32"),
        # the exact value that estimates are judged against
        dict(name="exact", kind="exact", side=4, bond=8, dtype="float32"),
        # training the selector's regressor: 32 features, 64 hidden units
        dict(name="train", kind="train", rows=32768, batch=4096, d_in=32, hidden=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["triangle", "batch", "batch", "torus", "torus", "ladder", "tree", "tree", "partial", "stream",
                       "exact", "train"])
    if kind == "triangle":
        return dict(kind=kind, count=_log_int(rng, 1, 64), n=rng.randint(17, 96), m=rng.choice([64, 256, 1024]),
                    samples=_log_int(rng, 4, 256), dtype=rng.choice(["float64", "float32"]),
                    graph=rng.random() < 0.3)
    if kind == "batch":
        m = rng.choice([256, 512, 1024, 1024, 2048])
        return dict(kind=kind, count=_log_int(rng, 24, 3000), m=m, samples=rng.randint(5, 24 * 1024 // max(m, 1024)),
                    dtype=rng.choice(["float32", "float32", "bfloat16"]),
                    dft=rng.choice(["bf16", "fft"]) if m == 1024 else "fft", tune=rng.random() < 0.5)
    if kind == "torus":
        m = rng.choice([512, 1024, 4096, 16384, 32768, 65536])
        bond = rng.randint(7, 16)
        most = (256 * 65536 * 32) // (bond ** 4 * 32) if m <= 4096 else 48 * 16384 // max(m, 16384)
        return dict(kind=kind, count=_log_int(rng, 1, min(128, most)), side=rng.choice([3, 4]), bond=bond, m=m,
                    samples=rng.randint(4, 32) if m <= 4096 else rng.randint(3, 12),
                    dtype=rng.choice(["float32", "float32", "bfloat16"]), tune=rng.random() < 0.5)
    if kind == "ladder":
        return dict(kind=kind, count=1, cores=rng.randint(6, 32), bond=rng.randint(20, 64), phys=rng.randint(20, 64),
                    m=rng.choice([1024, 4096]), samples=_log_int(rng, 8, 64), dtype="float32",
                    tune=rng.random() < 0.5)
    if kind == "tree":
        dtype = rng.choice(["float32", "float32", "float64"])
        return dict(kind=kind, count=rng.randint(1, 6), cores=rng.randint(4, 24), bond=rng.randint(13, 64),
                    phys=rng.randint(11, 64), m=rng.choice([512, 1024, 4096]), samples=_log_int(rng, 50, 1500),
                    dtype=dtype, products="f64" if dtype == "float64" else rng.choice(["f64", "f32", "f32", "bf16"]))
    if kind == "partial":
        return dict(kind=kind, bond=rng.randint(4, 9), m=rng.choice([256, 512, 1024]), samples=rng.randint(2, 8),
                    dtype=rng.choice(["float32", "bfloat16"]))
    if kind == "stream":
        return dict(kind=kind, vertices=rng.randint(200, 1024), edges=_log_int(rng, 2000, 32768),
                    m=rng.choice([1024, 4096, 8192]), samples=_log_int(rng, 8, 64),
                    dtype=rng.choice(["float32", "float64"]))
    if kind == "exact":
        side = rng.choice([3, 4])
        return dict(kind=kind, side=side, bond=rng.randint(3, 8), dtype=rng.choice(["float32", "float64"]))
    return dict(kind=kind, rows=rng.randint(5000, 32768), batch=rng.choice([1000, 2048, 4096]),
                d_in=rng.randint(16, 40), hidden=rng.choice([32, 64]))


# ---------------------------------------------------------------------------
# Networks: structure (orders, mode sizes, contracted mode pairs) and data.
# ---------------------------------------------------------------------------
def _random_structure(rng):
    """A random connected network with a cycle: a spanning tree plus 1 to p / 2 more contractions between tensors
    not yet joined, at most four modes per tensor, bonds U{2..32}, at most 2^18 entries per tensor."""
    while True:
        p = rng.randint(3, 12)
        pairs, degree = [], [0] * p
        for i in range(1, p):
            j = rng.choice([k for k in range(i) if degree[k] < 4])
            pairs.append((j, i))
            degree[i] += 1
            degree[j] += 1
        more = rng.randint(1, p // 2)
        free = [(a, b) for a in range(p) for b in range(a + 1, p) if (a, b) not in pairs]
        rng.shuffle(free)
        for a, b in free:
            if more and degree[a] < 4 and degree[b] < 4:
                pairs.append((a, b))
                degree[a] += 1
                degree[b] += 1
                more -= 1
        bonds = [rng.randint(2, 32) for _ in pairs]
        modes = [[(e, side) for e, ab in enumerate(pairs) for side in (0, 1) if ab[side] == k] for k in range(p)]
        if more or max(math.prod(bonds[e] for e, _ in mk) for mk in modes) > 1 << 18:
            continue
        where = {es: u for u, es in enumerate(es for mk in modes for es in mk)}
        return ([len(mk) for mk in modes], [bonds[e] for mk in modes for e, _ in mk],
                [(where[e, 0], where[e, 1]) for e in range(len(pairs))])


def _torus(side, bond):
    modes = lambda r, c: 4 * ((r % side) * side + c % side)  # noqa: E731  left, right, up, down
    edges = [e for r in range(side) for c in range(side)
             for e in ((modes(r, c) + 1, modes(r, c + 1)), (modes(r, c) + 3, modes(r + 1, c) + 2))]
    return [4] * side ** 2, [bond] * (4 * side ** 2), edges


def _train_shapes(cores, bond, phys):
    return [(phys, bond)] + [(bond, phys, bond)] * (cores - 2) + [(bond, phys)]


def _ladder(cores, bond, phys):
    shapes = _train_shapes(cores, bond, phys) * 2
    off = [0]
    for s in shapes:
        off.append(off[-1] + len(s))
    edges = [(off[b + k + 1] - 1, off[b + k + 1]) for b in (0, cores) for k in range(cores - 1)]
    edges += [(off[k] + (k > 0), off[cores + k] + (k > 0)) for k in range(cores)]
    return [len(s) for s in shapes], [n for s in shapes for n in s], edges


def _tree(cores, bond, phys):
    shapes = _train_shapes(cores, bond, phys) + [(phys,)] * cores
    off = [0]
    for s in shapes:
        off.append(off[-1] + len(s))
    edges = [(off[k + 1] - 1, off[k + 1]) for k in range(cores - 2)] + [(off[cores - 1] - 1, off[cores - 1])]
    edges += [(off[k] + (k > 0), off[cores + k]) for k in range(cores)]
    return [len(s) for s in shapes], [n for s in shapes for n in s], edges


@functools.lru_cache(maxsize=8)
def _structures(kind, count, *sizes):
    if kind == "batch":
        return [_random_structure(random.Random(7919 * i + 4)) for i in range(count)]
    if kind in ("triangle", "stream"):
        return [([2, 2, 2], [sizes[0]] * 6, [(1, 2), (3, 4), (0, 5)])] * count
    if kind == "torus":
        return [_torus(*sizes)] * count
    if kind == "partial":
        orders, dims, edges = _torus(3, sizes[0])
        return [(orders, dims, edges[2:])]
    return [(_ladder if kind == "ladder" else _tree)(*sizes)] * count


def _networks(case):
    kind = case["kind"]
    if kind == "torus" or kind == "exact":
        return _structures("torus", case.get("count", 1), case["side"], case["bond"])
    if kind in ("ladder", "tree"):
        return _structures(kind, case["count"], case["cores"], case["bond"], case["phys"])
    size = {"triangle": "n", "stream": "vertices", "partial": "bond"}.get(kind)
    return _structures(kind, case.get("count", 1), *([case[size]] if size else []))


def _shapes(structure):
    orders, dims, _ = structure
    out, u = [], 0
    for q in orders:
        out.append(tuple(dims[u:u + q]))
        u += q
    return out


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _data(case, seed):
    """Per network its device tensors: N(0, 1); U[0, 1) for the lattices; N(0, 1/64) for the tensor trains."""
    nets = _networks(case)
    shapes = [_shapes(s) for s in nets]
    # one allocation, each tensor at a multiple of 512 bytes as separate ones would be
    pad = 512 // ESIZE[case["dtype"]]
    sizes = [[math.prod(s) for s in net] for net in shapes]
    total = sum(-(-n // pad) * pad for net in sizes for n in net)
    if case["kind"] in ("torus", "exact"):
        flat = torch.rand(total, generator=_generator(seed), device="cuda")
    else:
        flat = torch.randn(total, generator=_generator(seed), device="cuda")
        if case["kind"] in ("ladder", "tree"):
            flat *= 0.125
    flat = flat.to(DTYPES[case["dtype"]])
    out, at = [], 0
    for net, ns in zip(shapes, sizes):
        ts = []
        for s, n in zip(net, ns):
            ts.append(flat[at:at + n].view(s))
            at += -(-n // pad) * pad
        out.append(ts)
    return nets, out


def _updates(case, seed):
    """Edge insertions of a directed graph with skewed endpoints, an eighth of them deleted again: the row-major
    matrix entries and their signs."""
    g, n, e = _generator(seed), case["vertices"], case["edges"]
    src, dst = ((torch.rand(e, generator=g, device="cuda", dtype=torch.float64) ** 2 * n).long().clamp_(max=n - 1)
                for _ in range(2))
    gone = torch.randperm(e, generator=g, device="cuda")[:e // 8]
    index = (src * n + dst)
    sign = torch.ones(e, dtype=torch.float64, device="cuda")
    return torch.cat([index, index[gone]]), torch.cat([sign, -sign[gone]])


def _features(case, seed):
    """Standardized features, a smooth target of them, and the regressor's first weights."""
    g, d, h, n = _generator(seed), case["d_in"], case["hidden"], case["rows"]
    X = torch.randn(n, d, generator=g, device="cuda")
    y = torch.tanh(X[:, 0] + 0.5 * X[:, 1] * X[:, 2]) + 0.3 * X[:, 3]
    parts = []
    for fan_out, fan_in, bias in ((h, d, h), (h, h, h), (1, h, 1)):
        a = math.sqrt(6.0 / (fan_in + fan_out))
        parts += [(2 * torch.rand(fan_out * fan_in, generator=g, device="cuda") - 1) * a,
                  torch.zeros(bias, device="cuda")]
    return X, y.contiguous(), torch.cat(parts)


LR = 2e-3


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        X, y, w = _features(case, seed)
        net = T.MLP(case["d_in"], case["hidden"], 0)
        net.set_params(w.cpu().numpy())
        return dict(kind=kind, net=net, X=X, y=y, batch=case["batch"])
    if kind == "stream":
        orders, dims, edges = _networks(case)[0]
        index, delta = _updates(case, seed)
        spec = T.NetworkSpec(orders, dims, edges, dtype=DTYPES[case["dtype"]])
        plan = T.Plan([spec], T.TN_CYCLIC, case["m"], case["samples"], seed % 1000, flags=T.TN_FLAG_RESIDENT)
        return dict(kind=kind, plan=plan, index=index, delta=delta, **_outputs(plan))
    nets, data = _data(case, seed)
    specs = [T.NetworkSpec(*s, tensors=ts) for s, ts in zip(nets, data)]
    if kind == "exact":
        return dict(kind=kind, spec=specs[0])
    if kind == "partial":
        plan = T.PartialPlan(specs[0], case["m"], case["samples"], seed % 1000)
    else:
        flags = T.TN_FLAG_AUTOTUNE if case.get("tune") else 0
        flags |= T.TN_FLAG_GRAPH if case.get("graph") else 0
        flags |= T.TN_FLAG_DFT_BF16 if case.get("dft") == "bf16" else 0
        flags |= {"f32": T.TN_FLAG_MFMA_F32, "bf16": T.TN_FLAG_MFMA_BF16}.get(case.get("products"), 0)
        plan = T.Plan(specs, T.TN_ACYCLIC if kind == "tree" else T.TN_CYCLIC, case["m"], case["samples"],
                      seed % 1000, flags=flags)
    return dict(kind="estimate", plan=plan, data=data, **_outputs(plan))


def _outputs(plan):
    return dict(stats=torch.empty(2 * plan.n_nets, dtype=torch.float64, device="cuda"),
                samples=torch.empty(plan.n_nets * plan.S, dtype=torch.float64, device="cuda"))


def run(state):
    kind = state["kind"]
    if kind == "exact":
        return T.tn_contract_exact(state["spec"])
    if kind == "train":
        losses = state["net"].train(state["X"], state["y"], batch=state["batch"], epochs=1, lr=LR)
        return {"losses": losses, "params": state["net"].params()}
    plan = state["plan"]
    if kind == "stream":  # every edge feeds the three matrices of tr(A A A)
        plan.reset()
        for k in range(3):
            plan.update(k, state["index"], state["delta"])
        plan.combine(state["stats"], state["samples"])
    else:
        plan.estimate(state["stats"], state["samples"])
    return {"stats": state["stats"], "samples": state["samples"]}


def work(case):
    """Inputs once, outputs once.  Operations: cyclic method S (sum of entries + p m log2 m) additions and
    butterflies; acyclic method 2 S entries per tensor with children (its product over the samples); the exact
    contraction its two joins of half-lattices and the rings that make them; training 6 per weight and row."""
    kind = case["kind"]
    if kind == "train":
        d, h, n = case["d_in"], case["hidden"], case["rows"]
        weights = h * d + h * h + 3 * h + 1
        return {"bytes": 4 * n * (d + 1) + 4 * weights * 2, "flops": 6 * n * weights}
    if kind == "stream":
        e = case["edges"] + case["edges"] // 8
        m, S = case["m"], case["samples"]
        return {"bytes": 16 * e + 8 * (S + 2), "flops": 3 * S * (2 * e + 2.5 * m * math.log2(m))}
    nets = _networks(case)
    sizes = [[math.prod(s) for s in _shapes(n)] for n in nets]
    entries = sum(sum(net) for net in sizes)
    moved = entries * ESIZE[case["dtype"]]
    if kind == "exact":
        b, side = case["bond"], case["side"]
        row = 2 * b ** (2 * side) * b ** 2 * 2  # a ring of `side` tensors closed on the row's 2 side legs
        return {"bytes": moved + 8, "flops": side * row + 2 * b ** (3 * side) * (side - 2)}
    S, m = case["samples"], case["m"]
    if kind == "tree":
        inner = sum(n for net in sizes for n in net if n > case["phys"])
        return {"bytes": moved + 8 * case["count"] * (S + 2), "flops": 2 * S * inner}
    out = case["bond"] ** 4 if kind == "partial" else case["count"]
    p = sum(len(net) for net in sizes)
    return {"bytes": moved + 8 * out * (S + 2), "flops": S * (2 * entries + 2.5 * p * m * math.log2(m))}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits.  The hash family (two-wise buckets, four-wise signs over 2^31 - 1, SplitMix64 keys) is
# the library's documented one; the cyclic method's spectra are taken as products with exp(-2 pi i j h / m).
# ---------------------------------------------------------------------------
def _mix(x):
    z = x + np.uint64(0x9E3779B97F4A7C15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _hashes(seeds, streams, S, n, m):
    """Buckets and signs of the streams (seeds[e], streams[e]) for samples 0 .. S - 1 at indices 0 .. n - 1, each of
    shape (streams, S, n)."""
    with np.errstate(over="ignore"):
        key = _mix(_mix(np.array(seeds, dtype=np.uint64))[:, None] ^ np.arange(S, dtype=np.uint64)[None, :])
        key = _mix(key ^ np.array(streams, dtype=np.uint64)[:, None])
        raw = [(_mix(key ^ np.uint64(i)) >> np.uint64(33)).astype(np.int64) for i in range(6)]
    raw = [torch.from_numpy(r).cuda()[:, :, None] for r in raw]
    i = torch.arange(n, device="cuda")
    h = ((1 + raw[1] % (P31 - 1)) * i + raw[0] % P31) % P31 % m
    v = raw[5] % P31
    for c in (raw[4], raw[3], raw[2]):
        v = (v * i + c % P31) % P31
    return h, 1.0 - 2.0 * (v & 1).double()


def _spectra(x, free, hs, signs, m, tw, J):
    """Spectra of the tensor sketches of x (FP64): shape (free assignments, S, J).  free: the free modes; hs, signs:
    per contracted mode its buckets (complement applied) and signs, each (S, n)."""
    order = free + [u for u in range(x.dim()) if u not in free]
    x = x.permute(order)
    F, dims = math.prod(x.shape[:len(free)]), x.shape[len(free):]
    S, split = hs[0].shape[0], (len(dims) + 1) // 2

    def phases(h, s, s0, s1):  # (S', indices of these modes, J) complex
        hh, ss = h[0][s0:s1], s[0][s0:s1]
        for a, b in zip(h[1:], s[1:]):
            hh = (hh[:, :, None] + a[s0:s1, None, :]).flatten(1)
            ss = (ss[:, :, None] * b[s0:s1, None, :]).flatten(1)
        j = torch.arange(J, device="cuda")
        return ss[:, :, None] * tw[(hh % m)[:, :, None] * j % m]

    R, L = math.prod(dims[:split]), math.prod(dims[split:])
    x = x.reshape(F, R, L)
    out = torch.empty(F, S, J, dtype=torch.complex128, device="cuda")
    step = max(1, (1 << 25) // (max(R * F, L, R) * J))
    for s0 in range(0, S, step):
        s1 = min(S, s0 + step)
        if split == len(dims):
            w = x.reshape(F, 1, R, 1).expand(F, s1 - s0, R, 1).to(torch.complex128)
        else:
            b = phases(hs[split:], signs[split:], s0, s1).permute(1, 0, 2).reshape(L, -1)
            flat = x.reshape(F * R, L)
            w = torch.complex(flat @ b.real.contiguous(), flat @ b.imag.contiguous())
            w = w.view(F, R, s1 - s0, J).permute(0, 2, 1, 3)
        out[:, s0:s1] = (phases(hs[:split], signs[:split], s0, s1) * w).sum(2)
    return out


def _cyclic(nets, data, m, S, seed):
    """Estimates (outputs, S) of Eq. (1): per network, or per entry of the output over its free modes."""
    J = m // 2 + 1
    k = torch.arange(m, device="cuda", dtype=torch.float64) * (2 * math.pi / m)
    tw = torch.complex(torch.cos(k), -torch.sin(k))
    wt = torch.full((J,), 2.0, dtype=torch.float64, device="cuda")
    wt[0] = 1.0
    wt[-1] = 1.0
    ids = [(seed + j, e) for j, (_, _, edges) in enumerate(nets) for e in range(len(edges))]
    widest = max(n for _, dims, _ in nets for n in dims)
    h_all, s_all = _hashes([a for a, _ in ids], [b for _, b in ids], S, widest, m)
    out, first = [], 0
    for (orders, dims, edges), ts in zip(nets, data):
        of = {u: (e, side) for e, uv in enumerate(edges) for side, u in enumerate(uv)}
        free_all = [u for u in range(len(dims)) if u not in of]
        prod, u0 = None, 0
        for q, x in zip(orders, ts):
            free = [u for u in range(q) if u0 + u not in of]
            hs, ss = [], []
            for u in range(q):
                if u not in free:
                    e, side = of[u0 + u]
                    h = h_all[first + e, :, :dims[u0 + u]]
                    hs.append((m - h) % m if side else h)
                    ss.append(s_all[first + e, :, :dims[u0 + u]])
            y = _spectra(x.double(), free, hs, ss, m, tw, J)
            if free_all:
                y = y.view(*[dims[u] if u - u0 in free else 1 for u in free_all], S, J)
            else:
                y = y[0]
            prod = y if prod is None else prod * y
            u0 += q
        first += len(edges)
        out.append(((prod.real * wt).sum(-1) / m).reshape(-1, S))
    return torch.cat(out)


def _acyclic(case, data, seed):
    """Estimates (networks, S) of Eq. (2) on the tree rooted at the first core, leaves to root."""
    cores, bond, phys, m, S = case["cores"], case["bond"], case["phys"], case["m"], case["samples"]
    out = []
    for j, ts in enumerate(data):
        ts = [t.double() for t in ts]
        seeds = seed + j
        legs, w = cores - 1, None  # contraction k joins cores k, k + 1; contraction cores - 1 + k core k and its vector
        for k in range(cores - 1, -1, -1):
            x = ts[k]
            h, s = _hashes([seeds], [legs + k], S, phys, m)
            slots = [(h[0], s[0], ts[cores + k].expand(S, phys))]
            if k < cores - 1:
                h, s = _hashes([seeds], [k], S, bond, m)
                slots.append((h[0], s[0], w))
                for d in (0, 1):  # the tensor sketch of the two children's buckets
                    th, tsn = _hashes([seeds], [(1 << 62) + (k << 32) + (2 << 16) + d], S, m, m)
                    h, s, v = slots[d]
                    slots[d] = (torch.gather(th[0], 1, h), s * torch.gather(tsn[0], 1, h), v)
                (h0, s0, v0), (h1, s1, v1) = slots
                b = ((h0[:, :, None] + h1[:, None, :]) % m).flatten(1)
                sg = (s0[:, :, None] * s1[:, None, :]).flatten(1)
                val = (v0[:, :, None] * v1[:, None, :]).flatten(1)
            else:
                b, sg, val = slots[0]
            r = torch.zeros(S, m, dtype=torch.float64, device="cuda").scatter_add_(1, b, sg * val)
            g = sg * torch.gather(r, 1, b)
            w = g @ x.reshape(bond if k else 1, -1).T
        out.append(w[:, 0])
    return torch.stack(out)


def _torus_value(ts, side):
    """The periodic lattice's value from its rows' transfer matrices."""
    b = ts[0].shape[0]
    total = None
    for r in range(side):
        a = ts[r * side].double()  # left, right, up, down -> left, right, (up), (down)
        a = a.reshape(b, b, b, b)
        for c in range(1, side):
            t = ts[r * side + c].double()
            lft, rgt, up, dn = a.shape
            a = torch.tensordot(a, t, dims=([1], [0])).permute(0, 3, 1, 4, 2, 5).reshape(lft, b, up * b, dn * b)
        row = torch.einsum("aaud->ud", a)
        total = row if total is None else total @ row
    return float(torch.trace(total))


def _trained(case, seed):
    X, y, w = _features(case, seed)
    X, y, w = X.double(), y.double(), w.double()
    d, h, n, batch = case["d_in"], case["hidden"], case["rows"], case["batch"]
    m1, m2, loss_sum = torch.zeros_like(w), torch.zeros_like(w), 0.0
    sizes = [h * d, h, h * h, h, h, 1]
    for t, r0 in enumerate(range(0, n, batch), start=1):
        w.requires_grad_(True)
        W1, b1, W2, b2, W3, b3 = torch.split(w, sizes)
        xb, yb = X[r0:r0 + batch], y[r0:r0 + batch]
        h1 = torch.tanh(xb @ W1.view(h, d).T + b1)
        h2 = torch.tanh(h1 @ W2.view(h, h).T + b2)
        sq = 0.5 * ((h2 @ W3 + b3 - yb) ** 2).sum()
        g, = torch.autograd.grad(sq / len(xb), w)
        loss_sum += float(sq)
        m1 = 0.9 * m1 + 0.1 * g
        m2 = 0.999 * m2 + 0.001 * g * g
        w = (w.detach() - LR * (m1 / (1 - 0.9 ** t)) / (torch.sqrt(m2 / (1 - 0.999 ** t)) + 1e-8))
    return {"losses": np.array([loss_sum / n]), "params": w.cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _trained(case, seed)
    if kind == "stream":
        n = case["vertices"]
        index, delta = _updates(case, seed)
        a = torch.zeros(n * n, dtype=torch.float64, device="cuda").index_add_(0, index, delta).view(n, n)
        est = _cyclic(_networks(case), [[a, a, a]], case["m"], case["samples"], seed % 1000)
    else:
        nets, data = _data(case, seed)
        if kind == "exact":
            return _torus_value(data[0], case["side"])
        if kind == "tree":
            est = _acyclic(case, data, seed % 1000)
        else:
            est = _cyclic(nets, data, case["m"], case["samples"], seed % 1000)
    stats = torch.stack([est.mean(1), est.var(1) if est.shape[1] > 1 else torch.zeros_like(est[:, 0])], 1)
    return {"stats": stats.reshape(-1), "samples": est.reshape(-1)}

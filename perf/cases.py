"""What a user of this library has it do, as cases that can be timed.

A case is one partition (its size, degrees, feature rows), a GraphSAGE sampler,
a prefetch buffer and the way the program drives the library; one pass is
`steps` minibatches from seeds to gathered feature rows, through the Python
binding:

  call "sample"   massive_sample and the round it owes, step by step
  call "async"    look-ahead, two batches in flight, as a training loop runs it
  call "noalloc"  massive_sample_noalloc (serving loops that may not allocate)

With an interval of `delta` steps a pass is one whole interval: `delta`
minibatches, then the eviction round owed by the last one. A delta of STATIC is
prefetching without eviction, and a pass is `steps` minibatches.

The partitions have the sizes of this repository's workloads (10K, 170K, 2.45M
and 111M nodes cut into 4, 8, 16 and 64 partitions). Their edges are drawn on
the GPU, so that the largest takes seconds: Chung-Lu degrees over the whole
graph, a random share of the nodes as the local ones, the halo as what their
edges reach, and a row's neighbours drawn in proportion to their own row
lengths, in ascending id.
"""
import math

import numpy as np
import torch

from paper_2410_22697_amd import Massive

STATIC = 100000  # no round within any run
DEPTH = 2        # batches in flight of a look-ahead loop
ROUNDS_BEFORE = 6

# one partition of a graph: the graph's nodes, mean degree and degree exponent,
# and the partition's local and halo nodes
GRAPHS = {
    "10k": dict(n=10_000, mean=10.0, beta=2.1, L=2500, H=5310),
    "170k": dict(n=170_000, mean=14.0, beta=2.2, L=21_250, H=86_096),
    "2m45": dict(n=2_450_000, mean=50.0, beta=2.0, L=153_125, H=1_446_105),
    "111m": dict(n=111_000_000, mean=29.0, beta=1.9, L=1_734_375, H=13_843_780),
}


def _case(graph, call, batch, fanout, d, dtype, pct, gamma, delta, steps, layout="rank"):
    c = dict(GRAPHS[graph]) if isinstance(graph, str) else dict(graph)
    f = list(fanout) + [0] * (4 - len(fanout))
    c.update(call=call, batch=batch, f1=f[0], f2=f[1], f3=f[2], f4=f[3], d=d, dtype=dtype, pct=pct, gamma=gamma,
             delta=delta, steps=steps, layout=layout)
    return c


def listed():
    return [
        # a serving loop's request: a few seeds, one minibatch at a time
        dict(name="serve_16_noalloc", **_case("170k", "noalloc", 16, (15, 10, 5), 128, "f32", 25, 0.95, STATIC, 1)),
        # the smallest training set-up, step by step, a round every eight steps
        dict(name="10k_interval_sync", **_case("10k", "sample", 256, (25, 10), 64, "f32", 25, 0.95, 8, 8)),
        # one minibatch of an arxiv-sized graph, waited for
        dict(name="170k_step_sync", **_case("170k", "sample", 1024, (15, 10, 5), 128, "f32", 25, 0.95, STATIC, 1)),
        # arxiv-sized training with look-ahead and eviction
        dict(name="170k_interval", **_case("170k", "async", 1024, (15, 10, 5), 128, "f32", 25, 0.95, 16, 16)),
        # a last batch of odd size, odd row width, two hops, bf16 rows
        dict(name="170k_ragged_bf16", **_case("170k", "async", 777, (7, 13), 50, "bf16", 35, 0.995, STATIC, 5)),
        # products-sized training, prefetching without eviction, half the halo buffered
        dict(name="2m45_static", **_case("2m45", "async", 2000, (15, 10, 5), 100, "f32", 50, 0.95, STATIC, 8)),
        # the paper's two-layer sampler and batch, with eviction
        dict(name="2m45_two_layer_interval", **_case("2m45", "async", 2000, (10, 25), 100, "f32", 25, 0.95, 32, 32)),
        # bf16 rows, large batches, a round every four steps over half the halo
        dict(name="2m45_bf16_stress", **_case("2m45", "async", 4096, (20, 15, 10), 100, "bf16", 50, 0.8, 4, 4)),
        # scores kept over every global id
        dict(name="2m45_gid_interval", **_case("2m45", "async", 1000, (15, 10, 5), 100, "f32", 25, 0.95, 16, 16, "gid")),
        # one of 64 partitions of a papers-sized graph: one minibatch waited for
        dict(name="111m_step_sync", **_case("111m", "sample", 1024, (15, 10, 5), 128, "f32", 25, 0.95, STATIC, 1)),
        # the same partition trained with look-ahead, prefetching without eviction
        dict(name="111m_static", **_case("111m", "async", 1024, (15, 10, 5), 128, "f32", 25, 0.95, STATIC, 8)),
        # and with eviction: the benchmark's workload
        dict(name="111m_interval", **_case("111m", "async", 1024, (15, 10, 5), 128, "f32", 25, 0.95, 32, 32)),
    ]


def draw(rng):
    """One more case between the smallest and the largest listed ones."""
    n = int(math.exp(rng.uniform(math.log(10_000), math.log(20_000_000))))
    parts = rng.randint(3, 8) if n < 500_000 else rng.randint(8, 32)
    g = dict(n=n, mean=round(rng.uniform(8, 50 if n < 5_000_000 else 25), 1), beta=round(rng.uniform(1.9, 2.3), 2))
    g["L"] = n // parts
    # a node outside the partition is in its halo if one of its edges leads into it
    w, du = _grid(n, g["beta"], g["mean"])
    g["H"] = min(n - g["L"] - 1, max(1000, int((n - g["L"]) * float((du * -np.expm1(-w / parts)).sum()))))
    hops = rng.choice([1, 2, 2, 3, 3])
    fanout = [rng.randint(5, 25), rng.randint(4, 20), rng.randint(3, 10)][:hops]
    batch = min(int(math.exp(rng.uniform(math.log(8), math.log(2500)))), g["L"] // 4)
    bound = batch
    for f in fanout:
        bound = min(g["L"] + g["H"], bound * (1 + f))
    call = rng.choice(["sample", "async", "async", "noalloc"])
    if call == "noalloc" and bound > 1_300_000:
        call = "sample"
    dtype = rng.choice(["f32", "f32", "bf16"])
    d = rng.randint(8, 128) * (1 if dtype == "f32" else 2)
    delta = rng.choice([4, 8, 16, 32, STATIC, STATIC])
    steps = delta if delta != STATIC else (1 if call != "async" else rng.randint(3, 8))
    return _case(g, call, batch, fanout, d, dtype, rng.choice([15, 25, 25, 35, 50, 60]),
                 rng.choice([0.8, 0.95, 0.995]), delta, steps, rng.choice(["rank", "rank", "rank", "gid"]))


def _fanout(case):
    return [case["f%d" % k] for k in range(1, 5) if case["f%d" % k]]


def _row_bytes(case):
    return case["d"] * (4 if case["dtype"] == "f32" else 2)


def _i0(n, beta, mean):
    """The offset that gives the degree law of _law its mean."""
    a, wmax = 1.0 / (beta - 1.0), math.sqrt(n * mean)
    u, du = _QUANTILES
    lo, hi = 1e-9, 1e9
    for _ in range(100):
        i0 = math.sqrt(lo * hi)
        m = float((wmax * ((u * n + i0) / i0) ** (-a) * du).sum())
        lo, hi = (lo, i0) if m > mean else (i0, hi)
    return i0


# 4096 quantiles of the nodes in order of degree, finer towards the hubs, and their weights
_QUANTILES = (((np.arange(4096) + 0.5) / 4096) ** 4, 4 * ((np.arange(4096) + 0.5) / 4096) ** 3 / 4096)


def _grid(n, beta, mean):
    """Degrees at the quantiles, and the quantiles' weights."""
    u, du = _QUANTILES
    i0 = _i0(n, beta, mean)
    return math.sqrt(n * mean) * ((u * n + i0) / i0) ** (-1.0 / (beta - 1.0)), du


def _law(n, beta, mean, device):
    """Chung-Lu expected degrees of n nodes, longest first:
    w_max ((i + i0) / i0)^(-1 / (beta - 1)) with w_max = sqrt(n mean)."""
    i0 = _i0(n, beta, mean)
    i = torch.arange(n, dtype=torch.float64, device=device) + 0.5
    return math.sqrt(n * mean) * ((i + i0) / i0) ** (-1.0 / (beta - 1.0))


def _partition(case, gen, device):
    """Row offsets (int64) and columns (int32) of one partition, on the device."""
    L, H, n = case["L"], case["H"], case["n"]
    R = L + H
    w = _law(n, case["beta"], case["mean"], device)
    total = float(w.sum())
    w = w[torch.randperm(n, generator=gen, device=device)]
    # the first L nodes are local; of the others, the H that an edge from them
    # reaches first (each after a time of rate w) are the halo
    reach = -torch.log1p(-torch.rand(n - L, generator=gen, device=device, dtype=torch.float64)) / w[L:]
    halo = torch.sort(torch.sort(reach).indices[:H]).values
    w = torch.cat([w[:L], w[L:][halo]])
    del reach, halo
    # a halo node's row holds only its neighbours in the partition's own view
    w[L:] *= float(w.sum()) / total
    deg = (w + torch.rand(R, generator=gen, device=device, dtype=torch.float64)).long().clamp_(min=1)
    indptr = torch.zeros(R + 1, dtype=torch.int64, device=device)
    torch.cumsum(deg, 0, out=indptr[1:])
    nnz = int(indptr[-1])
    # stubs[x]: the row of entry x; entry j of a row of length d takes the stub
    # at a random place of the j-th of d equal parts of them
    stubs = torch.repeat_interleave(torch.arange(R, dtype=torch.int32, device=device), deg)
    cols = torch.empty(nnz, dtype=torch.int32, device=device)
    chunk = 1 << 27
    for lo in range(0, nnz, chunk):
        hi = min(nnz, lo + chunk)
        row = stubs[lo:hi].long()
        at = torch.arange(lo, hi, device=device, dtype=torch.float64) - indptr[row]
        at += torch.rand(hi - lo, generator=gen, device=device, dtype=torch.float64)
        at *= nnz
        at /= deg[row]
        cols[lo:hi] = stubs[at.long().clamp_(max=nnz - 1)]
    return indptr, cols, deg


def _host(x, pinned=False):
    """x's values in host memory."""
    h = torch.empty(x.shape, dtype=x.dtype, pin_memory=pinned)
    h.copy_(x)
    return h


def _rows(n, case, gen, device, out):
    """n feature rows, N(0, 1), into the host tensor `out` (uint8 [n, row bytes])."""
    d, dt = case["d"], torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    chunk = max(1, (1 << 27) // d)
    for lo in range(0, n, chunk):
        hi = min(n, lo + chunk)
        out[lo:hi].copy_(torch.randn(hi - lo, d, generator=gen, device=device).to(dt).view(torch.uint8))


class State:
    """A training loop's own objects: the context, its batches, its seeds."""

    def __init__(self, case, seed):
        dev = "cuda"
        gen = torch.Generator(device=dev)
        gen.manual_seed(seed)
        L, H, rb = case["L"], case["H"], _row_bytes(case)
        indptr, cols, deg = _partition(case, gen, dev)
        # the largest arrays through pinned memory, which the GPU copies to and from at full rate
        h_indptr, h_cols = _host(indptr), _host(cols, pinned=True)
        h_deg = _host(deg[L:])
        gid = torch.sort(torch.randperm(case["n"], generator=gen, device=dev)[:H]).values.int() if case["n"] < 1 << 25 \
            else (torch.arange(H, device=dev, dtype=torch.int64) * case["n"] // H).int()
        h_gid = _host(gid)
        del indptr, cols, deg, gid
        store = torch.empty((H, rb), dtype=torch.uint8, pin_memory=True)
        _rows(H, case, gen, dev, store)
        local = torch.empty((L, rb), dtype=torch.uint8, pin_memory=True)
        _rows(L, case, gen, dev, local)
        self.gm = Massive(L, H, h_indptr.numpy(), h_cols.numpy(), h_gid.numpy(), h_deg.numpy(), local, store, rb,
                          _fanout(case), case["pct"], case["gamma"], case["delta"], seed & 0xFFFFFFFF,
                          score_layout=case["layout"], n_global=case["n"])
        del h_cols, local
        torch.cuda.empty_cache()
        self.case = case
        self.batches = [self.gm.alloc_batch(case["batch"]) for _ in range(DEPTH if case["call"] == "async" else 1)]
        for bb in self.batches:
            for x in [bb.nodes, bb.mask, bb.feat] + bb.indptr + bb.indices:
                x.zero_()
        # an epoch's shuffled seeds, in batches; the run goes round them
        n_sets = max(1, min(64, L // case["batch"]))
        order = torch.randperm(L, generator=gen, device=dev)[:n_sets * case["batch"]].int()
        self.seeds = list(order.reshape(n_sets, case["batch"]).unbind(0))
        self.t = 0
        self.outs = None
        if case["delta"] != STATIC:
            # the run is some rounds in (the first ones swing, as the buffer moves
            # away from the initial one) and one step past the last of them, so
            # that a pass is an interval with its round at the end
            cap = max(self.gm.cap, 1)
            self.outs = tuple(torch.zeros(cap, dtype=torch.int32, device=dev) for _ in range(3))
            for _ in range(1 + ROUNDS_BEFORE * case["delta"]):
                self.gm.sample(self.next_seeds(), self.batches[0])
                self.gm.evict_step(wait=False)

    def next_seeds(self):
        s = self.seeds[self.t % len(self.seeds)]
        self.t += 1
        return s


def prepare(case, seed):
    return State(case, seed)


def _batch_outputs(bb):
    """A batch's buffers, as they are sized (its rows and edges are the first of them)."""
    return [bb.nodes, bb.mask, bb.feat, bb.indptr, bb.indices]


def run(state):
    gm, case = state.gm, state.case
    call, steps = case["call"], case["steps"]
    sizes, held = [], {}
    if call == "async":
        flying = []

        def finish():
            bb = flying.pop(0)
            r = gm.wait(bb)
            sizes.append(r.n + r.e + [r.local, r.hits, r.misses])
            held[id(bb)] = bb

        for i in range(steps):
            bb = state.batches[i % DEPTH]
            gm.sample_async(state.next_seeds(), bb)
            flying.append(bb)
            if i + 1 < steps or state.outs is None:
                gm.evict_step(wait=False)
                if len(flying) == DEPTH:
                    finish()
        k = gm.evict_step(out=state.outs) if state.outs is not None else 0
        while flying:
            finish()
    else:
        bb = state.batches[0]
        step = gm.sample if call == "sample" else gm.sample_noalloc
        for i in range(steps):
            r = step(state.next_seeds(), bb)
            sizes.append(r.n + r.e + [r.local, r.hits, r.misses])
            if i + 1 < steps or state.outs is None:
                gm.evict_step(wait=False)
        k = gm.evict_step(out=state.outs) if state.outs is not None else 0
        held[id(bb)] = bb
    # every step's sizes and class counts, the batches still held, the round's sets
    out = [np.array(sizes, np.int64), [_batch_outputs(bb) for bb in held.values()]]
    if state.outs is not None:
        out += [k, list(state.outs)]
    return out


def _expected(case):
    """Expected frontier rows n_0..n_K, sampled edges e_1..e_K and keys drawn
    (row lengths of the rows longer than the fanout) of one minibatch. A
    neighbour is drawn in proportion to its row length, so after E draws a
    node of length w is in the frontier with probability 1 - exp(-E w / S)."""
    L, n = case["L"], case["n"]
    w, du = _grid(n, case["beta"], case["mean"])
    c_lo, c_hi = 1e-12, 1e6  # the halo's size fixes how far its nodes are reached
    for _ in range(100):
        c = math.sqrt(c_lo * c_hi)
        size = float((du * -np.expm1(-c * w)).sum()) * (n - L)
        c_lo, c_hi = (c_lo, c) if size > case["H"] else (c, c_hi)
    halo = du * -np.expm1(-c * w) * (n - L)
    view = (float((w * du).sum()) * L + float((w * halo).sum())) / (float((w * du).sum()) * n)
    count = np.concatenate([du * L, halo])
    w = np.maximum(np.concatenate([w, w * view]), 1.0)
    S = float((w * count).sum())
    seeds = np.zeros_like(w)
    seeds[:len(du)] = case["batch"] / L
    ns, es, keys, E = [float(case["batch"])], [], 0.0, 0.0
    p = seeds
    for f in _fanout(case):
        rows = p * count
        e = float((rows * np.minimum(w, f)).sum())
        keys += float((rows * np.where(w > f, w, 0.0)).sum())
        es.append(e)
        E += e
        p = 1.0 - (1.0 - seeds) * np.exp(-E * w / S)
        ns.append(float((p * count).sum()))
    return ns, es, keys


def work(case):
    """Of one pass. Bytes: every input row read and written once; per frontier
    row its two offsets, id, mask and output offset; per sampled edge the
    column read and the position written; a round reads each score and writes
    what it changes. Operations: a Philox4x32-10 block (20 multiplies, 40
    exclusive ors, 20 adds) gives four keys."""
    ns, es, keys = _expected(case)
    rb = _row_bytes(case)
    rows = ns[-1] * (2 * rb + 4 + 1 + 16) + sum(ns[:-1]) * 4 + sum(es) * 8
    total = rows * case["steps"]
    if case["delta"] != STATIC:
        cap = case["H"] * case["pct"] // 100
        total += 4 * case["H"] + 12 * cap
    return {"bytes": total, "flops": keys * 20 * case["steps"]}


def tolerance(case):
    """Ids, offsets, masks and copied bytes: the same whatever the implementation."""
    return "exact"


def exact(case, seed):
    """No output is a computed floating-point number (rows are copied bit by bit)."""
    return None

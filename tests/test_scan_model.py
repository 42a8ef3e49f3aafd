"""A model of the single-pass scans (decoupled look-back): tiles start in order
(block order or tickets) but run in any interleaving, each publishes its
aggregate and then its inclusive prefix in one 64-bit word, and waits by reading
the words of the tiles before it, a window at a time. Two forms:

- the seeds' and the rounds' scans (lookback_exclusive): one wave reads 64
  predecessors at a time; words tagged with the launch's epoch, so that an older
  epoch's are not ready;
- the frontier's (fr_lookback): all NT threads of the block read NT predecessors
  at a time, wave by wave; two 31-bit sums in one word, state 1 or 2 in its top
  bits, the words cleared before the launch.

The model checks that every tile gets the exact exclusive prefixes and that the
run ends. A tile publishes its aggregate some time after it starts, so a
successor can find its word not ready and must wait. It restates the kernels'
steps; the GPU tests exercise the kernels."""
import random

import pytest

WAVE = 64


def run_model(ntiles, seed, start_prob=0.3):
    rnd = random.Random(seed)
    epoch = 5
    t_agg, t_inc = 2 * epoch, 2 * epoch + 1
    flags = [((2 * 3 + 1) << 32) | rnd.randrange(1000) for _ in range(ntiles)]  # an older epoch's flags
    agg = [rnd.randrange(0, 5000) for _ in range(ntiles)]
    state, started, result = {}, [], {}
    pending = list(range(ntiles))
    for _ in range(10_000_000):
        if len(result) == ntiles:
            break
        if pending and (not started or rnd.random() < start_prob):
            b = pending.pop(0)  # blocks start in order
            state[b] = None     # computing its aggregate: its flag is still an older epoch's
            started.append(b)
            continue
        live = [b for b in started if b not in result]
        if not live:
            continue
        b = rnd.choice(live)
        if state[b] is None:  # the aggregate is ready: publish it, then look back
            flags[b] = ((t_inc if b == 0 else t_agg) << 32) | agg[b]
            state[b] = [b - 1, 0]
            continue
        p, excl = state[b]
        done = p < 0
        if not done:
            vals = [flags[p - lane] if p - lane >= 0 else (t_inc << 32) for lane in range(WAVE)]
            tags = [f >> 32 for f in vals]
            ready = [t in (t_agg, t_inc) for t in tags]
            inc = [t == t_inc for t in tags]
            k = inc.index(True) if any(inc) else WAVE - 1
            if all(ready[:k + 1]):
                excl += sum(v & 0xFFFFFFFF for v in vals[:k + 1])
                if any(inc):
                    done = True
                else:
                    p -= WAVE
                    done = p < 0
            state[b] = [p, excl]
        if done:
            if b > 0:
                flags[b] = (t_inc << 32) | (excl + agg[b])
            result[b] = excl
    assert len(result) == ntiles, "the model did not finish"
    want = 0
    for b in range(ntiles):
        assert result[b] == want, (ntiles, seed, b)
        want += agg[b]


@pytest.mark.parametrize("ntiles", [1, 2, 3, 63, 64, 65, 129, 300])
def test_lookback_exclusive_prefixes(ntiles):
    for seed in range(10):
        run_model(ntiles, seed)


def fr_state(st, n, e):
    assert 0 <= n < 1 << 31 and 0 <= e < 1 << 31
    return st << 62 | e << 31 | n


def run_frontier(ntiles, NT, seed, most, start_prob=0.3):
    rnd = random.Random(seed)
    agg = [(rnd.randrange(most), rnd.randrange(most)) for _ in range(ntiles)]
    flags, state, result, pending = [0] * ntiles, {}, {}, list(range(ntiles))
    for _ in range(10_000_000):
        if len(result) == ntiles:
            break
        if pending and (not state or rnd.random() < start_prob):
            state[pending.pop(0)] = None
            continue
        live = [b for b in state if b not in result]
        if not live:
            continue
        b = rnd.choice(live)
        if state[b] is None:
            flags[b] = fr_state(2 if b == 0 else 1, *agg[b])
            state[b] = [b - 1, 0, 0]
            continue
        p, n, e = state[b]
        if p >= 0:
            add, st_all = [0, 0], 1
            for w in range(NT // WAVE):  # (a wave after one that is not ready, or that ends, does not count)
                if st_all != 1:
                    break
                f = [flags[p - w * WAVE - x] if p - w * WAVE - x >= 0 else fr_state(2, 0, 0) for x in range(WAVE)]
                sts = [v >> 62 for v in f]
                k = sts.index(2) if 2 in sts else WAVE - 1
                st_all = 0 if not all(sts[:k + 1]) else 2 if 2 in sts else 1
                if st_all:
                    add[0] += sum(v & 0x7FFFFFFF for v in f[:k + 1])
                    add[1] += sum(v >> 31 & 0x7FFFFFFF for v in f[:k + 1])
            if st_all:
                n, e = n + add[0], e + add[1]
                p = -1 if st_all == 2 else p - NT
            state[b] = [p, n, e]
        if p < 0:
            if b > 0:
                flags[b] = fr_state(2, n + agg[b][0], e + agg[b][1])
            result[b] = (n, e)
    assert len(result) == ntiles, "the model did not finish"
    want = [0, 0]
    for b in range(ntiles):
        assert result[b] == tuple(want), (ntiles, NT, seed, b)
        want = [x + y for x, y in zip(want, agg[b])]


@pytest.mark.parametrize("ntiles,NT", [(1, 256), (2, 256), (65, 256), (257, 256), (300, 256), (600, 512)])
def test_frontier_lookback_of_two_sums(ntiles, NT):
    for seed in range(4):
        run_frontier(ntiles, NT, seed, 65536)
    run_frontier(ntiles, NT, 9, (1 << 31) // ntiles)  # the largest sums

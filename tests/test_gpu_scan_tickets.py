"""Scans whose blocks take their tiles by ticket (launches above the block-order
limit; here the limit is 0, so that every scan takes them, one-tile ones too):
the counters go back to zero after each launch, whatever the launch before it
was, so every step and round below starts from a fresh one. Each step and round
against the oracle, with refused seeds, no-alloc and look-ahead steps between."""
import numpy as np
import pytest

from gpu_util import compare_state, compare_step, log, make_gpu, require_gpu, run_parity, to_dev
from helpers import Problem, workload_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(monkeypatch):
    require_gpu()
    monkeypatch.setenv("MASSIVE_ORDERED_WAVES", "0")


@pytest.mark.parametrize("name", ["cl10k", "cl170k"])
def test_steps(name):
    from paper_2410_22697_amd import MassiveError
    prob, sched, w = workload_problem(name, delta=2)
    K = len(prob.fanout)
    orc, gm = prob.oracle(), make_gpu(prob)
    bbs = [gm.alloc_batch(w.batch) for _ in range(2)]
    for t in range(0, 8, 2):
        log("%s tickets t=%d" % (name, t))
        with pytest.raises(MassiveError):
            gm.sample(to_dev(np.array([3, 3], np.int32)), bbs[0])
        pair = [sched.seeds(t), sched.seeds(t + 1)[:1 + 5 * t]]
        if t % 4:
            res = []
            for s, bb in zip(pair, bbs):
                res.append(gm.sample_noalloc(to_dev(s), bb))
                gm.evict_step(wait=False)
        else:
            for s, bb in zip(pair, bbs):
                gm.sample_async(to_dev(s), bb)
                gm.evict_step(wait=False)
            res = [gm.wait(bb) for bb in bbs]
        for i, s in enumerate(pair):
            st = orc.sample(s)
            orc.evict_step()
            compare_step("t=%d" % (t + i), st, res[i], bbs[i], K)
    compare_state("end", orc, gm)


@pytest.mark.parametrize("layout", ["rank", "gid"])
def test_rounds(layout):
    # a halo of three tiles, a buffer above the one-block sort
    H, L, d = 11000, 300, 60
    rng = np.random.default_rng(3)
    col = (H * rng.random((L, d)) ** 3).astype(np.int32) + L
    indptr = np.minimum(np.arange(L + H + 1, dtype=np.int64), L) * d
    feats = rng.standard_normal((L + H, 2)).astype(np.float32)
    prob = Problem(L, H, indptr, col.reshape(-1), rng.permutation(3 * H)[:H].astype(np.int32),
                   rng.integers(1, 50, H).astype(np.int64), feats[:L], feats[L:], 2, "f32", (40,), 60, 0.5, 1)
    seeds = [rng.permutation(L)[:150].astype(np.int32) for _ in range(4)]
    gm = make_gpu(prob, score_layout=layout, n_global=3 * H)
    rounds, _, _ = run_parity("tickets %s" % layout, prob, lambda t: seeds[t], 4, gm=gm)
    assert rounds >= 2

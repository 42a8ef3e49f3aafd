"""Eviction rounds where their launches change: buffers of 4096 slots and one
more (the one-block sort against the digit passes), halos that are and are not
whole tiles, more evictions than candidates (the narrowing's three sorts), and
score ties across the threshold; a round after every step, every set and score
against the oracle, with S_A by rank and by global id."""
import numpy as np
import pytest

from gpu_util import make_gpu, require_gpu, run_parity
from helpers import Problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _problem(H, pct, fanout, gamma):
    """300 local nodes with 60 halo neighbours each, drawn unevenly so that
    scores range from many ties to single large counts."""
    rng = np.random.default_rng(H + pct)
    L, d = 300, 60
    col = (H * rng.random((L, d)) ** 3).astype(np.int32) + L
    indptr = np.minimum(np.arange(L + H + 1, dtype=np.int64), L) * d
    feats = rng.standard_normal((L + H, 2)).astype(np.float32)
    return Problem(L, H, indptr, col.reshape(-1), rng.permutation(3 * H)[:H].astype(np.int32),
                   rng.integers(1, 50, H).astype(np.int64), feats[:L], feats[L:], 2, "f32", fanout, pct, gamma, 1)


@pytest.mark.parametrize("layout", ["rank", "gid"])
@pytest.mark.parametrize("H,pct", [(8192, 50), (8194, 50), (4096, 25), (4099, 100), (5000, 80), (20000, 20), (13, 40)])
def test_round_every_step(H, pct, layout):
    prob = _problem(H, pct, (40,), 0.5)
    rng = np.random.default_rng(pct)
    seeds = [rng.permutation(prob.L)[:150 if H > 100 else 0].astype(np.int32) for _ in range(6)]
    gm = make_gpu(prob, score_layout=layout, n_global=3 * H)
    rounds, _, _ = run_parity("rounds H=%d pct=%d %s" % (H, pct, layout), prob, lambda t: seeds[t], 6, gm=gm)
    assert rounds >= (0 if pct == 100 else 4 if H > 100 else 1)


@pytest.mark.parametrize("layout", ["rank", "gid"])
@pytest.mark.parametrize("H,pct", [(2, 50), (3, 34), (3, 67), (4, 50), (5, 40)])
def test_round_of_the_smallest_halos(H, pct, layout):
    # score arrays below and just above one 16-byte vector
    prob = _problem(H, pct, (40,), 0.5)
    prob.halo_gid = np.arange(H, dtype=np.int32)[::-1].copy()
    gm = make_gpu(prob, score_layout=layout, n_global=H)
    assert gm.cap >= 1
    seeds = [np.arange(t, dtype=np.int32) for t in (0, 0, 3, 0, 0)]
    run_parity("rounds H=%d pct=%d %s" % (H, pct, layout), prob, lambda t: seeds[t], 5, gm=gm)

"""The sampler's ways of choosing from a row, at the row lengths and fanouts
where one ends and the next begins: whole rows, rows of one Philox iteration
(256 positions), rows filtered by one wave, long rows by one wave or by a whole
block (above 2048), and the candidate lists of one quad, two quads and single
keys per lane (fanouts up to 18, up to 56 and above). Both samplers: the one
for small frontiers and the one-wave-per-row one (a frontier bound above
65,536 rows). First thresholds that let far too many keys through (the list
overflows and the search comes back down) or hardly any (it goes up first) are
forced, as usual ones hardly ever do either. Everything is compared element by
element with the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, run_parity
from helpers import Problem

pytestmark = pytest.mark.gpu

LENGTHS = (1, 2, 17, 18, 19, 20, 55, 56, 57, 58, 59, 63, 64, 65, 128, 253, 255, 256, 257, 260, 511, 512, 513, 1000, 2047,
           2048, 2049, 4100, 20001)


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _problem(R, fanout, hubs=1400):
    """Nodes below `hubs` have the lengths above in turn, the others three
    neighbours; nine neighbours of ten are below `hubs`."""
    rng = np.random.default_rng(len(fanout) * 1000 + fanout[-1])
    deg = np.full(R, 3, np.int64)
    deg[:hubs] = np.resize(LENGTHS, hubs)
    indptr = np.zeros(R + 1, np.int64)
    np.cumsum(deg, out=indptr[1:])
    far = rng.integers(0, R, indptr[-1], dtype=np.int32)
    near = rng.integers(0, hubs, indptr[-1], dtype=np.int32)
    indices = np.where(rng.random(indptr[-1]) < 0.9, near, far).astype(np.int32)
    L, H = hubs, R - hubs
    feats = np.arange(R, dtype=np.float32).reshape(R, 1)
    return Problem(L, H, indptr, indices, np.arange(H, dtype=np.int32), deg[L:].copy(), feats[:L], feats[L:], 1, "f32",
                   fanout, 25, 0.9, 2, seed=fanout[-1])


@pytest.mark.parametrize("fo", [1, 2, 5, 17, 18, 19, 33, 55, 56, 57, 58, 100])
def test_small_frontier(fo):
    prob = _problem(5000, (fo,))
    rng = np.random.default_rng(fo)
    seeds = [rng.permutation(prob.L)[:700].astype(np.int32) for _ in range(3)]
    run_parity("rows fo=%d" % fo, prob, lambda t: seeds[t], 3, state_every=3)


@pytest.mark.parametrize("fo", [3, 18, 19, 55, 56, 57, 58])
def test_wave_per_row(fo):
    prob = _problem(140000, (100, fo))
    rng = np.random.default_rng(fo)
    seeds = [rng.permutation(prob.L)[:n].astype(np.int32) for n in (700, 1350)]
    run_parity("rows by waves fo=%d" % fo, prob, lambda t: seeds[t], 2, state_every=2)


@pytest.mark.parametrize("keys", [0.5, 300, 4000])
@pytest.mark.parametrize("fo", [5, 18, 19, 56, 57])
def test_first_threshold_far_off(monkeypatch, fo, keys):
    # `keys` expected survivors of the first threshold: below the fanout, above
    # what the lists hold, and all of most rows; by rows of a wave, of a block
    # (above 256 here) and of a wave of many
    monkeypatch.setenv("MASSIVE_FIRST_KEYS", str(keys))
    monkeypatch.setenv("MASSIVE_BIG_ROW", "256" if fo % 2 else "1500")
    rng = np.random.default_rng(fo)
    prob = _problem(5000, (fo,))
    seeds = rng.permutation(prob.L)[:700].astype(np.int32)
    run_parity("rows fo=%d first keys %s" % (fo, keys), prob, lambda t: seeds, 1)
    prob = _problem(140000, (100, fo))
    seeds = rng.permutation(prob.L)[:700].astype(np.int32)
    run_parity("rows by waves fo=%d first keys %s" % (fo, keys), prob, lambda t: seeds, 1)

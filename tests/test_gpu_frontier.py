"""The frontier scan (new nodes in order, their rows and offsets) at its edges:
id spaces on and beside the edges of its bitmap tiles and of its choice of
tile, local counts at word edges, and runs of consecutive new ids that fill
whole tiles, many times the rows a block holds at once. Everything is compared
element by element with the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, run_parity
from helpers import Problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _runs_problem(L, R, active, length, stride, fanout):
    """Rows of the first `active` nodes hold `length` consecutive ids from
    v * stride on (mod R); the others are empty."""
    indptr = np.minimum(np.arange(R + 1, dtype=np.int64), active) * length
    first = np.arange(active, dtype=np.int64) * stride
    indices = ((first[:, None] + np.arange(length)) % R).astype(np.int32).reshape(-1)
    H = R - L
    feats = np.arange(R, dtype=np.float32).reshape(R, 1)
    return Problem(L, H, indptr, indices, np.arange(H, dtype=np.int32), (indptr[L + 1:] - indptr[L:-1]).astype(np.int64),
                   feats[:L], feats[L:], 1, "f32", fanout, 25, 0.9, 2)


@pytest.mark.parametrize("L,R", [
    (40, 64), (64, 2048), (33, 2049), (2048, 4095),      # one and two of the smallest tiles
    (1000, 12288 * 32), (1024, 12288 * 32 + 1),          # either side of the middle tile size
    (1000, 16384 * 32), (1024, 16384 * 32 + 1),
    (1000, 131072 * 32), (1023, 131072 * 32 + 33)])      # either side of the largest
def test_tile_edges(L, R):
    prob = _runs_problem(L, R, min(R, 40000), 60, 37, (60, 60) if R > 5000 else (60, 7))
    rng = np.random.default_rng(R)
    seeds = [rng.permutation(L)[:n].astype(np.int32) for n in (min(L, 500), 1, 0, min(L, 300))]
    run_parity("tiles L=%d R=%d" % (L, R), prob, lambda t: seeds[t], len(seeds), state_every=3)


def test_every_id_is_local():
    prob = _runs_problem(4096, 4096, 4096, 50, 3, (50, 5))
    seeds = [np.arange(k, 4096, 5, dtype=np.int32) for k in range(3)]
    run_parity("no halo, id space on a word edge", prob, lambda t: seeds[t], 3)

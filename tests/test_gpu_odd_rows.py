"""The miss gather where rows and 16-byte vectors do not line up: every row of
a store that starts 0, 4, 8 or 12 bytes past a 16-byte boundary and ends right
behind its last row, read over the host link (no buffer) and, with rounds,
written through into refilling slots; each step against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, run_parity, make_gpu
from helpers import tiny_problem, workload_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _offset_store(prob, offset):
    import torch
    flat = np.ascontiguousarray(prob.halo_store).view(np.uint8).reshape(-1)
    t = torch.empty(offset + flat.size, dtype=torch.uint8, pin_memory=True)[offset:]
    assert t.data_ptr() % 16 == offset
    t.copy_(torch.from_numpy(flat))
    return t


@pytest.mark.parametrize("offset", [0, 4, 8, 12])
@pytest.mark.parametrize("d,dtype", [(1, "f32"), (3, "f32"), (5, "f32"), (25, "f32"), (50, "f32"), (257, "f32"),
                                     (4, "f32"), (300, "bf16")])
def test_every_row(d, dtype, offset):
    # each halo node is some local node's neighbour, and the fanout takes whole rows
    prob = tiny_problem(n_local=40, n_halo=60, p=0.3, seed=d, d=d, fanout=(120, 2), buffer_pct=0, dtype=dtype)
    seeds = np.arange(prob.L, dtype=np.int32)
    _, _, misses = run_parity("d=%d offset=%d" % (d, offset), prob, lambda t: seeds, 2,
                              gm=make_gpu(prob, store=_offset_store(prob, offset)))
    assert misses == 2 * prob.H


@pytest.mark.parametrize("d,offset", [(50, 0), (50, 8), (25, 4)])
def test_refilling_slots(d, offset):
    prob, sched, w = workload_problem("cl10k", d=d, dtype="f32", delta=1, gamma=0.9)
    rounds, _, _ = run_parity("cl10k d=%d offset=%d" % (d, offset), prob, sched.seeds, 6, buffer_rows_every=1,
                              gm=make_gpu(prob, store=_offset_store(prob, offset)))
    assert rounds >= 4

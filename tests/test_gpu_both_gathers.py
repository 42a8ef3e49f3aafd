"""Both gathers in one launch: steps whose two lists are of very different
lengths in turn (a single seed, then a whole batch, and back), in look-ahead and
waited for, with a small, a usual and a whole buffer; each against the oracle."""
import numpy as np
import pytest

from gpu_util import compare_state, compare_step, log, make_gpu, require_gpu, to_dev
from helpers import workload_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("pct,delta", [(0, 1000), (25, 3), (97, 4), (100, 1000)])
def test_uneven_steps(pct, delta):
    prob, sched, w = workload_problem("cl170k", buffer_pct=pct, delta=delta)
    K = len(prob.fanout)
    orc, gm = prob.oracle(), make_gpu(prob)
    bbs = [gm.alloc_batch(w.batch) for _ in range(2)]
    flying = []

    def finish():
        t, bb, seeds = flying.pop(0)
        res = gm.wait(bb)
        st = orc.sample(seeds)
        orc.evict_step()
        compare_step("pct=%d t=%d n0=%d" % (pct, t, len(seeds)), st, res, bb, K)

    for t in range(9):
        n0 = (1, w.batch, 0, w.batch, 2, 300, w.batch, 1, w.batch)[t]
        log("both gathers pct=%d t=%d n0=%d" % (pct, t, n0))
        if len(flying) == 2 or t % 4 == 3:
            while flying:
                finish()
        seeds = sched.seeds(t)[:n0]
        bb = bbs[t % 2]
        if t % 4 == 3:  # waited for
            res = gm.sample(to_dev(seeds), bb)
            gm.evict_step(wait=False)
            st = orc.sample(seeds)
            orc.evict_step()
            compare_step("pct=%d t=%d n0=%d" % (pct, t, n0), st, res, bb, K)
        else:
            gm.sample_async(to_dev(seeds), bb)
            gm.evict_step(wait=False)
            flying.append((t, bb, seeds))
    while flying:
        finish()
    compare_state("end", orc, gm)

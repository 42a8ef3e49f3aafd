"""Steps that are waited for at once (both gathers in one launch on the main
stream) between look-ahead steps, no-alloc steps, rounds with refills in
flight, refused seeds and timed steps, in every order that the slots' cleared
sizes and the events of earlier steps can meet; each step against the oracle."""
import numpy as np
import pytest

from gpu_util import compare_state, compare_step, log, make_gpu, require_gpu, to_dev
from helpers import workload_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("d,dtype,delta", [(64, "f32", 3), (5, "f32", 100000), (6, "f32", 2), (50, "bf16", 4)])
@pytest.mark.parametrize("seed", [0, 1])
def test_mixed_steps(d, dtype, delta, seed):
    from paper_2410_22697_amd import MAX_INFLIGHT, MassiveError
    prob, sched, w = workload_problem("cl10k", d=d, dtype=dtype, delta=delta)
    K = len(prob.fanout)
    orc, gm = prob.oracle(), make_gpu(prob)
    rng = np.random.default_rng(seed)
    bbs = [gm.alloc_batch(w.batch) for _ in range(MAX_INFLIGHT)]
    flying, t = [], 0

    def finish():
        u, bb, seeds = flying.pop(0)
        res = gm.wait(bb)
        st = orc.sample(seeds)
        orc.evict_step()
        compare_step("t=%d" % u, st, res, bb, K)

    while t < 40:
        kind = rng.choice(["async", "async", "sample", "sample", "noalloc", "bad", "timed"])
        seeds = sched.seeds(t)[: int(rng.integers(0, w.batch + 1))]
        log("d=%d t=%d %s n0=%d in flight %d" % (d, t, kind, len(seeds), len(flying)))
        if kind == "timed":
            gm.set_timing(bool(rng.integers(2)))
            continue
        if kind == "noalloc" or kind == "bad" or len(flying) == MAX_INFLIGHT:
            while flying:
                finish()
        bb = bbs[t % MAX_INFLIGHT]
        if kind == "bad":
            with pytest.raises(MassiveError):
                gm.sample(to_dev(np.append(seeds, [3, 3]).astype(np.int32)[-w.batch:]), bb)
            continue
        if kind == "async":
            gm.sample_async(to_dev(seeds), bb)
            flying.append((t, bb, seeds))
            gm.evict_step(wait=False)
        else:
            res = (gm.sample if kind == "sample" else gm.sample_noalloc)(to_dev(seeds), bb)
            gm.evict_step(wait=bool(rng.integers(2)))
            out = (t, res, bb, seeds)
            while flying:
                finish()
            st = orc.sample(seeds)
            orc.evict_step()
            compare_step("t=%d" % t, st, out[1], bb, K)
        t += 1
    while flying:
        finish()
    compare_state("end", orc, gm)
    assert np.array_equal(gm.buffer_rows(), orc.buffer_rows())

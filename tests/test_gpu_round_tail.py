"""Late preemptive rounds, whose cull and refinement also score the next round
when a plan has few live hypotheses: hypothesis counts around the list length
from which they do, draws around a workgroup's share, one tree to sixteen, more
modes per draw than a lane loads ahead, and refinement off. The trace equals the
oracle's, and the results equal those of the same attempt in a batch too large
for it."""
import numpy as np
import pytest

import synthroom as sr
from tests.gpu_util import banner, need_gpu, pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


@pytest.mark.parametrize("hyps,draws,trees,modes,refine", [
    (2, 64, 5, 10, 1), (3, 17, 5, 10, 1), (5, 64, 1, 4, 1), (33, 1, 3, 10, 1), (64, 8, 5, 10, 1), (65, 15, 5, 10, 1),
    (66, 16, 4, 10, 0), (127, 500, 5, 10, 1), (129, 33, 9, 10, 1), (200, 100, 16, 32, 1), (300, 130, 5, 50, 1),
    (1024, 497, 2, 50, 1)])
def test_late_rounds(dev, hyps, draws, trees, modes, refine):
    import oracle
    import paper_1801_08361_amd as rl
    banner(f"late rounds N={hyps} B={draws} T={trees} M={modes} refine={refine}")
    pp, po = pair(n_trees=trees, depth=7, reservoir_size=128, max_modes=modes, n_hypotheses=hyps, batch_pixels=draws,
                  min_cluster=1 if modes > 10 else 8, refine=refine)
    g, o = rl.Forest(pp), oracle.Forest(po)
    sc = sr.small_scene(91, 200, 150)
    for k in range(8):
        d, c = sc.render_adapt(k)
        g.adapt_frame(*to_dev(d, c, dev), sc.K, sc.adapt_poses[k])
        o.adapt(d, c, sc.K, sc.adapt_poses[k])
    per = max(1, hyps >> 5) * ((draws + 15) // 16)     # workgroups of a late round, at least
    for q in (2, 6):
        d0, c0 = sc.render_query(q)
        d, c = to_dev(d0, c0, dev)
        for rep in range(2):                           # the second run's buffers hold the first's values
            got = g.relocalise_ex(d, c, sc.K, seed=40 + q)
            t = g.trace(hyps)
        so, _, sco, to = o.relocalise(d0, c0, sc.K, seed=40 + q, trace=True)
        assert got["status"] == so and np.array_equal(t["hyp_try"], to["hyp_try"])
        if so != 0:
            continue
        n = int(to["n_rounds"][0])
        assert got["n_rounds"] == n and np.array_equal(t["n_alive"][:n], to["n_alive"][:n])
        for r in range(n):
            na = int(to["n_alive"][r])
            assert np.array_equal(t["alive"][r, :na], to["alive"][r, :na]), r
            np.testing.assert_allclose(t["energy"][r, :na], to["energy"][r, :na], rtol=1e-4, atol=1e-4)
        assert got["final_hyp"] == to["final_hyp"][0] and abs(got["score"] - sco) < 1e-6
        copies = min(2 + 1024 // per, 300)
        res = rl.Batch(tune=False).run([dict(forest=g, depth=d, rgb=c, K=sc.K, seed=40 + q)] * copies)
        for b in (res[0], res[-1]):
            for k in ("status", "n_rounds", "final_hyp", "score", "mode_evals", "pair_evals"):
                assert b[k] == got[k], k
            assert np.array_equal(b["pose"], got["pose"])

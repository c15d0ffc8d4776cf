"""Hypothesis generation at the sizes where its mode colour rows change: one
16-byte load and its remainders, rows of up to three loads and of blocks of
four, 32-bit and 64-bit masks, single trees and many, and tries that fill less
or more than one wavefront. The tries found equal the oracle's, and a
checkpoint holds the plain colours of the modes."""
import numpy as np
import pytest

import synthroom as sr
from tests.gpu_util import banner, need_gpu, pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


@pytest.mark.parametrize("modes,trees,tries,tol", [
    (1, 5, 64, 15), (4, 3, 64, 20), (5, 5, 65, 15), (8, 2, 64, 30), (12, 5, 100, 15), (13, 5, 64, 15), (16, 1, 64, 40),
    (17, 5, 7, 25), (28, 4, 64, 15), (32, 16, 64, 2), (33, 3, 130, 15), (49, 5, 1, 60), (64, 8, 64, 254), (10, 16, 64, 0)])
def test_rows(dev, tmp_path, modes, trees, tries, tol):
    import oracle
    import paper_1801_08361_amd as rl
    banner(f"hypotheses M={modes} T={trees} tries={tries} tol={tol}")
    pp, po = pair(n_trees=trees, depth=6, reservoir_size=128, max_modes=modes, n_hypotheses=96, batch_pixels=32,
                  max_tries=tries, rgb_tol=tol, min_cluster=1)
    g, o = rl.Forest(pp), oracle.Forest(po)
    sc = sr.small_scene(81, 160, 120)
    for k in range(6):
        d, c = sc.render_adapt(2 * k)
        g.adapt_frame(*to_dev(d, c, dev), sc.K, sc.adapt_poses[2 * k])
        o.adapt(d, c, sc.K, sc.adapt_poses[2 * k])
    path = str(tmp_path / "forest.bin")
    g.update_modes()
    g.drop_reservoirs()
    g.save(path)
    got = [g.modes(t, 0, g.L) for t in range(g.T)]
    stride = (modes + 3) // 4 * 4
    want = np.full((g.T, g.L, stride), 0xFFFFFFFF, np.uint32)
    for t, (m, n) in enumerate(got):
        used = np.arange(modes)[None, :] < n[:, None]
        want[t, :, :modes][used] = (m["rgb"][used].astype(np.uint32) << np.arange(0, 24, 8, dtype=np.uint32)).sum(1)
    raw = np.fromfile(path, np.uint32)
    leaf_inputs = g.T * g.L * 16                 # the section after the colour rows, the file's last
    assert np.array_equal(raw[-leaf_inputs - want.size:-leaf_inputs], want.ravel())
    loaded = rl.Forest.load(path)
    for q in (1, 5):
        d, c = sc.render_query(q)
        _, _, _, to = o.relocalise(d, c, sc.K, seed=70 + q, n_hyp=96, trace=True)
        for f in (g, loaded):
            f.relocalise(*to_dev(d, c, dev), sc.K, seed=70 + q, n_hyp=96)
            tg = f.trace(96)
            assert np.array_equal(tg["hyp_try"], to["hyp_try"]), q
            ok = to["hyp_try"] >= 0
            np.testing.assert_allclose(tg["hyp_pose"][ok], to["hyp_pose"][ok], atol=1e-9)

"""Modes of many leaves at the reservoir size where they stop being handed out in
turn (64 points) and start being handed out by a ticket (more), with more leaves
than workgroups. Every leaf's modes equal the oracle's."""
import numpy as np
import pytest

import synthroom as sr
from tests.gpu_util import assert_modes_equal, banner, need_gpu, pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


@pytest.mark.parametrize("reservoir,min_cluster", [(1, 1), (4, 0), (16, 1), (63, 0), (64, 1), (65, 1), (65, 0)])
def test_many_leaves(dev, reservoir, min_cluster):
    import torch

    import oracle
    import paper_1801_08361_amd as rl
    pp, po = pair(n_trees=3, depth=11, reservoir_size=reservoir, max_modes=6, min_cluster=min_cluster)
    g, o = rl.Forest(pp), oracle.Forest(po)
    K, rng = sr.intrinsics(240, 180), np.random.default_rng(reservoir)
    banner(f"modes of many leaves R={reservoir} min_cluster={min_cluster}")
    for k in range(2):
        # depths in steps and random colours: pixels spread over the leaves, points close together
        d = torch.from_numpy((1500 + 20 * rng.integers(0, 8, size=(180, 240))).astype(np.uint16))
        c = torch.from_numpy(rng.integers(0, 256, size=(180, 240, 3)).astype(np.uint8))
        pose = np.eye(4)
        pose[0, 3] = 0.3 * k
        g.adapt_frame(*to_dev(d, c, dev), K, pose)
        o.adapt(d, c, K, pose)
        changed = 0
        for t in range(g.T):
            changed += int((g.counters(t) > 0).sum())
            mg, ng = g.modes(t, 0, g.L)
            for leaf in range(g.L):
                mo = o.leaf_modes(t, leaf)
                assert ng[leaf] == len(mo), (k, t, leaf)
                assert_modes_equal(mg[leaf][: ng[leaf]], mo.view(mg.dtype) if len(mo) else mg[leaf][:0])
        assert changed > 2048   # workgroups of the mode kernel

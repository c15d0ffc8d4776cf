"""Split training's level kernels at the sizes where they change: sample counts
around a unit and a scan block, nodes of one unit and of several, the three
sharings of a unit by wavefronts, empty nodes, frames whose planes need
padding, and frames of several sizes. Sums are integers, so the nodes equal
the oracle's."""
import numpy as np
import pytest

import synthroom as sr
from tests.gpu_util import banner, need_gpu, pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def train_both(dev, sc, frames, stride, n_cand, extra=(), **kw):
    """Nodes of the GPU's and the oracle's training on frames [(depth, rgb,
    pose)]; `extra` GPU frames hold no valid pixel."""
    import oracle
    import paper_1801_08361_amd as rl
    pp, po = pair(reservoir_size=4, max_modes=4, **kw)
    g, o = rl.Forest(pp), oracle.Forest(po)
    g.train([(*to_dev(d, c, dev), sc.K, T) for d, c, T in frames] + list(extra), stride, n_cand)
    o.train([(d.numpy(), c.numpy(), T) for d, c, T in frames], sc.K, stride, n_cand)
    return g.nodes(), o.nodes()


def equal(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


# samples: one; around a wavefront, the small unit (256) and the large one
# (512); several units and scan blocks; each with nodes that stay empty
@pytest.mark.parametrize("keep,depth", [(1, 4), (63, 3), (64, 6), (255, 1), (256, 5), (257, 5), (511, 3), (512, 3),
                                        (513, 4), (1025, 9), (2049, 12), (19000, 8)])
def test_sample_counts(dev, keep, depth):
    import torch
    sc = sr.small_scene(83, 161, 119)
    d, c = sc.render_adapt(3)
    flat = d.numpy().reshape(-1).copy()
    valid = np.flatnonzero((flat >= 500) & (flat <= 5000))
    assert len(valid) >= keep
    flat[valid[keep:]] = 0
    banner(f"train samples={keep} depth={depth}")
    g, o = train_both(dev, sc, [(torch.from_numpy(flat.reshape(d.shape)), c, sc.adapt_poses[3])], 1, 64, n_trees=2, depth=depth)
    assert equal(g, o)


def test_no_samples(dev):
    import torch
    sc = sr.small_scene(83, 33, 17)
    d, c = sc.render_adapt(0)
    banner("train without samples")
    g, o = train_both(dev, sc, [(torch.zeros_like(d), c, sc.adapt_poses[0])], 2, 5, n_trees=3, depth=4)
    assert equal(g, o)


# the same samples with a frame of another size and focal length beside them
# (which holds none) take the kernels that look every frame up
@pytest.mark.parametrize("depth", [3, 8, 12])
def test_frames_of_several_sizes(dev, depth):
    import torch
    sc = sr.small_scene(84, 163, 121)
    frames = [(*sc.render_adapt(k), sc.adapt_poses[k]) for k in (0, 7)]
    other = (torch.zeros((50, 71), dtype=torch.uint16, device=dev), torch.zeros((50, 71, 3), dtype=torch.uint8, device=dev),
             sr.intrinsics(71, 50), sc.adapt_poses[1])
    banner(f"train several sizes depth={depth}")
    g, o = train_both(dev, sc, frames, 2, 33, extra=[other], n_trees=2, depth=depth)
    assert equal(g, o)

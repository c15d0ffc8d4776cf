"""Adaptation at the sizes where the ranks change their chunk: 2048, 4096 or 8192
pixels by the pixels over all trees, on both sides of each switch, with full and
ragged last chunks, in the deepest trees, and in one forest frame after frame;
and the prefix over chunks on both sides of the share a wavefront holds in
registers (24 of four wavefronts' 96). Counters and entries equal the oracle's."""
import numpy as np
import pytest

import synthroom as sr
from tests.gpu_util import banner, need_gpu, pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def chunk_of(T, P, L):
    """pixels per chunk, as the library chooses them"""
    e = 4 if L > 32768 else 8
    while e > 2 and T * P < 160 * 1024 * e:
        e //= 2
    return 1024 * e


def adapt_both(dev, sizes, **kw):
    import oracle
    import paper_1801_08361_amd as rl
    pp, po = pair(max_modes=4, **kw)
    g, o = rl.Forest(pp), oracle.Forest(po)
    for k, (w, h) in enumerate(sizes):
        sc = sr.small_scene(73, w, h)
        d, c = sc.render_adapt(3 * k)
        g.adapt_frame(*to_dev(d, c, dev), sc.K, sc.adapt_poses[3 * k])
        o.adapt(d, c, sc.K, sc.adapt_poses[3 * k])
        for t in range(g.T):
            cnt = g.counters(t)
            used = np.flatnonzero(cnt)
            if g.L <= 4096:
                want = np.array([o.reservoir(t, leaf)[1] for leaf in range(g.L)])
                assert np.array_equal(cnt, want), (k, t)
            some = used[np.linspace(0, len(used) - 1, min(len(used), 200)).astype(int)]
            busiest = used[np.argsort(cnt[used])[::-1][:64]]
            for leaf in np.union1d(some, busiest):
                eg, ng = g.reservoir(t, int(leaf))
                eo, no = o.reservoir(t, int(leaf))
                assert int(ng[0]) == no, (k, t, leaf)
                m = min(no, g.R)
                assert np.array_equal(eg[0][:m], eo[:m]), (k, t, leaf)


# (trees, width, height, pixels per chunk, chunks)
SIZES = [(5, 362, 362, 2048, 64), (5, 512, 256, 4096, 32), (5, 331, 396, 4096, 33),
         (5, 511, 513, 4096, 64), (5, 512, 512, 8192, 32), (5, 513, 512, 8192, 33)]


@pytest.mark.parametrize("trees,width,height,chunk,chunks", SIZES)
def test_chunk_sizes(dev, trees, width, height, chunk, chunks):
    P = width * height
    assert chunk_of(trees, P, 1 << 7) == chunk and -(-P // chunk) == chunks
    banner(f"adapt {trees} trees {width}x{height}")
    adapt_both(dev, [(width, height)] * 2, n_trees=trees, depth=7, reservoir_size=32)


@pytest.mark.parametrize("depth,width,height,chunk", [(16, 331, 396, 4096), (16, 513, 512, 4096), (15, 513, 512, 8192),
                                                      (1, 513, 512, 8192)])
def test_depths(dev, depth, width, height, chunk):
    assert chunk_of(5, width * height, 1 << depth) == chunk
    banner(f"adapt depth={depth} {width}x{height}")
    adapt_both(dev, [(width, height)], n_trees=5, depth=depth, reservoir_size=8)


# 96 chunks, 97 (one wavefront's share is 25) and 100 (each one's is)
@pytest.mark.parametrize("width,height,chunks", [(384, 512, 96), (443, 444, 97), (640, 320, 100)])
def test_prefix_shares(dev, width, height, chunks):
    assert -(-width * height // chunk_of(1, width * height, 1 << 7)) == chunks
    banner(f"adapt {chunks} chunks")
    adapt_both(dev, [(width, height)] * 2, n_trees=1, depth=7, reservoir_size=64)


def test_sizes_in_one_forest(dev):
    """large, small and ragged frames by turns: the smaller one has more chunks"""
    banner("adapt frames of many sizes")
    adapt_both(dev, [(512, 512), (362, 362), (64, 1), (331, 396), (513, 512)], n_trees=5, depth=7, reservoir_size=32)

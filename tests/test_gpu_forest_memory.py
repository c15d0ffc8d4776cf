"""Device memory kept from destroyed forests goes back to the device on request,
so that any other allocator of the process can have it, and the next forest
takes it back in time; a new forest in another's memory shows nothing of it, in
its mode slots and in its checkpoint."""
import numpy as np
import pytest

import synthroom as sr
from tests.gpu_util import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def test_trim_gives_everything_back(dev):
    import torch
    import paper_1801_08361_amd as rl
    p = rl.params_default(n_trees=16, depth=13, reservoir_size=1024, max_modes=10)
    rl.Forest(p).close()   # what the runtime itself keeps is there before the first reading
    rl.trim()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    banner("two forests of 2.8 GB, created and destroyed")
    fs = [rl.Forest(p) for _ in range(2)]
    assert torch.cuda.mem_get_info()[0] < free0 - (4 << 30)
    for f in fs:
        f.close()
    rl.trim()
    # 64 MB is the runtime's own granularity; a reservoir table has 2 GB
    assert torch.cuda.mem_get_info()[0] >= free0 - (64 << 20)
    rl.trim()
    f = rl.Forest(p)
    assert f.memory() > 2 << 30
    f.close()
    rl.trim()
    assert torch.cuda.mem_get_info()[0] >= free0 - (64 << 20)


def test_new_forest_is_empty_where_another_was(dev, tmp_path):
    import paper_1801_08361_amd as rl
    sc = sr.small_scene(107, 200, 150)
    # a table of modes of 2 MB and one of 40 KB
    for kw in (dict(n_trees=4, depth=10, reservoir_size=32), dict(n_trees=2, depth=4, reservoir_size=64)):
        banner(f"forest after another {kw}")
        p = rl.params_default(max_modes=10, min_cluster=1, **kw)
        files = []
        for k in range(2):
            f = rl.Forest(p)
            for t in range(f.T):
                m, n = f.modes(t, 0, f.L)
                assert not n.any() and not m.view(np.uint8).any()
            d, c = sc.render_adapt(5)
            g = to_dev(d, c, dev)
            # the second one has a tenth of the frame
            h = 150 if k == 0 else 15
            f.adapt_frame(g[0][:h].contiguous(), g[1][:h].contiguous(), sc.K, sc.adapt_poses[5])
            for t in range(f.T):
                m, n = f.modes(t, 0, f.L)
                assert n.any()
                past = np.arange(f.M)[None, :] >= n[:, None]
                assert not m[past].view(np.uint8).any()
            f.save(str(tmp_path / f"{k}"))
            files.append((tmp_path / f"{k}").read_bytes())
            f.close()
        # the same frame into a forest that follows another: the same file
        f = rl.Forest(p)
        f.adapt_frame(g[0][:15].contiguous(), g[1][:15].contiguous(), sc.K, sc.adapt_poses[5])
        f.save(str(tmp_path / "again"))
        assert (tmp_path / "again").read_bytes() == files[1]
        f.close()

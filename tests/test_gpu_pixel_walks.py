"""Per-pixel inputs and labels for the numbers of trees that walk together and
their remainders, shallow and deep trees, leaves with none to many modes, and
outputs that are not 16-byte aligned, against the oracle."""
import ctypes as C

import numpy as np
import pytest

import synthroom as sr
from tests.gpu_util import banner, need_gpu, pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


@pytest.mark.parametrize("trees,depth,modes,width,height", [
    (1, 1, 1, 64, 48), (2, 10, 3, 161, 121), (3, 4, 5, 100, 75), (4, 12, 4, 129, 97), (5, 10, 10, 160, 120),
    (6, 7, 9, 90, 70), (7, 3, 17, 80, 60), (9, 9, 6, 75, 61), (16, 6, 32, 96, 72)])
def test_walks(dev, trees, depth, modes, width, height):
    import oracle
    import torch
    import paper_1801_08361_amd as rl
    banner(f"pixel walks T={trees} D={depth} M={modes} {width}x{height}")
    pp, po = pair(n_trees=trees, depth=depth, reservoir_size=64, max_modes=modes, min_cluster=2)
    g, o = rl.Forest(pp), oracle.Forest(po)
    sc = sr.small_scene(111, width, height)
    for k in range(4):
        d, c = sc.render_adapt(2 * k)
        g.adapt_frame(*to_dev(d, c, dev), sc.K, sc.adapt_poses[2 * k])
        o.adapt(d, c, sc.K, sc.adapt_poses[2 * k])
    d, c = sc.render_query(2)
    d = d.clone()
    d[5:20, 7:30] = 0                                      # invalid pixels among the asked ones
    rng = np.random.default_rng(trees)
    pix = rng.integers(0, width * height, size=777).astype(np.int32)
    dd, dc = to_dev(d, c, dev)
    px = torch.from_numpy(pix).to(dev)
    x, xf = rl.pixel_features(g, dd, dc, sc.K, px, with_fp32=True)
    ref = o.features24(d.numpy(), c.numpy(), sc.K, pix)
    exact = [k for k in range(24) if k not in (10, 11, 12, 14, 15, 16, 18, 19, 20)]
    assert np.array_equal(xf.cpu().numpy()[:, exact], ref[:, exact])
    np.testing.assert_allclose(xf.cpu().numpy(), ref, rtol=2e-6, atol=1e-7)
    # the same values to places that are only as aligned as their type
    L = rl.lib()
    K = rl.reloc_intrinsics(width, height, *(float(k) for k in sc.K))
    xo = torch.zeros(777 * 32 + 1, dtype=torch.int16, device=dev)
    fo = torch.zeros(777 * 24 + 1, dtype=torch.float32, device=dev)
    rc = L.reloc_pixel_features(g.handle, dd.data_ptr(), dc.data_ptr(), C.byref(K), px.data_ptr(), 777,
                                xo[1:].data_ptr(), fo[1:].data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    assert torch.equal(xo[1:].view(777, 32), x) and torch.equal(fo[1:].view(777, 24), xf)
    for pose in (sc.query_poses[2], sc.adapt_poses[0]):
        y = rl.label_pixels(g, dd, dc, sc.K, pose, px).cpu().numpy()
        assert np.array_equal(y, o.label(d.numpy(), c.numpy(), sc.K, pose, pix))

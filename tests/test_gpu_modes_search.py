"""The tiled neighbour search of the mode kernel and its plain fallback against
the oracle: point counts around the tile, group and sort sizes, points that all
coincide or tie, padded negative coordinates, and the extents and radii at
which the kernel changes from one search to the other. Densities, parents,
clusters and sums are integers, so modes agree bit for bit (kappa's logarithms
to 1e-6)."""
import numpy as np
import pytest

from tests.gpu_util import assert_modes_equal, banner, need_gpu, pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def clustered(rng, n, extent, spread):
    """n points around a dozen centres in a box of the given extent, with a
    few strays and repeated points, on whole millimetres."""
    centres = rng.integers(0, extent + 1, size=(12, 3))
    xyz = centres[rng.integers(0, 12, size=n)] + rng.integers(-spread, spread + 1, size=(n, 3))
    stray = rng.random(n) < 0.1
    xyz[stray] = rng.integers(0, extent + 1, size=(int(stray.sum()), 3))
    again = rng.random(n) < 0.05
    xyz[again] = xyz[0]
    return np.clip(xyz, 0, extent)


def check(xyz, rng, **kw):
    import oracle
    import paper_1801_08361_amd as rl
    pp, po = pair(reservoir_size=1024, max_modes=10, **kw)
    g = rl.Forest(pp)
    p = np.zeros(len(xyz), dtype=rl.ENTRY_DTYPE)
    p["x"], p["y"], p["z"] = xyz.T
    p["r"], p["g"], p["b"] = rng.integers(0, 256, size=(3, len(xyz)))
    mg = g.modes_from_points(p)
    mo, _ = oracle.modes_from_points(po, p)
    assert_modes_equal(mg, mo.view(mg.dtype) if len(mo) else mg[:0])
    return len(mo)


@pytest.mark.parametrize("n", [1, 3, 7, 8, 9, 63, 64, 65, 72, 127, 128, 129, 255, 256, 257, 320, 511, 512, 513, 777,
                               1023, 1024])
def test_point_counts(dev, n):
    rng = np.random.default_rng(n)
    banner(f"modes search n={n}")
    found = check(clustered(rng, n, 6000, 90) - 2500, rng, min_cluster=1)
    assert found > 0


# the widest axis just inside, at and past 28 m, and coordinates far from zero
@pytest.mark.parametrize("extent", [0, 15, 2032, 2033, 27999, 28000, 28001, 60000])
@pytest.mark.parametrize("offset", [0, -1_000_000])
def test_extents(dev, extent, offset):
    rng = np.random.default_rng(extent + 1)
    xyz = clustered(rng, 600, extent, min(80, extent))
    xyz[1] = 0
    xyz[2] = extent
    banner(f"modes search extent={extent} offset={offset}")
    assert check(xyz + offset, rng, min_cluster=3) > 0


# radii 0, equal, swapped, and around the 2 m at which the search changes
@pytest.mark.parametrize("rd,rl", [(0, 0), (0, 100), (50, 50), (300, 100), (1999, 2000), (2000, 2000), (2001, 100),
                                   (50, 2001), (20000, 20000)])
def test_radii(dev, rd, rl):
    rng = np.random.default_rng(rd + rl)
    banner(f"modes search radii {rd} {rl}")
    assert check(clustered(rng, 500, 9000, 400), rng, min_cluster=1, dens_radius_mm=rd, link_radius_mm=rl) > 0


# lattices: many equal densities and equal distances, decided by the index
@pytest.mark.parametrize("step", [1, 25, 50, 100])
def test_ties(dev, step):
    rng = np.random.default_rng(step)
    xyz = rng.integers(0, 9, size=(1000, 3)) * step
    banner(f"modes search lattice {step}")
    assert check(xyz, rng, min_cluster=2) > 0

"""Road top-K where a distance bin decides: bins of one to many points, exact ties, and a cut
bin that just fits the staging buffer or just does not."""
import numpy as np
import pytest

from tests.test_parity_edge_gpu import _params, _sim
from tests._parity import compare_obs, oracle_for
from tests._util import tiny_world

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("obs_road", [1, 2])
@pytest.mark.parametrize("over", [-4, -3, -2, 0, 3])
@pytest.mark.parametrize("K", [1, 3, 66, 200])
def test_cut_bin_at_the_staging_limit(gpu, oracle_mod, K, over, obs_road):
    """K - 1 points on a spiral, then one point repeated: the K-th bin holds all the copies, and
    the staged points number stage + over, where stage = K + 60 up to a multiple of 4.  The
    keys of the copies are equal, so their indices decide; indices are compared exactly and
    features with compare_obs's bounds."""
    stage = (K + 60 + 3) // 4 * 4
    copies = stage + over - (K - 1)
    r = 3.0 + 17.0 * np.arange(K - 1) / max(K - 1, 1)
    th = 2.4 * np.arange(K - 1)
    pts = list(zip(r * np.cos(th), r * np.sin(th)))
    rng = np.random.default_rng(100 * K + over + 4)
    pts = [pts[i] for i in rng.permutation(K - 1)]
    for i in rng.integers(0, len(pts) + 1, copies):
        pts.insert(int(i), (24.0, 7.0))
    road = [(x, y, 0.1, 0 | 256) for x, y in pts]
    sc = tiny_world([(0.0, 0.0, 0.3, 4.5, 2.0)], extra_road=road, params=_params(top_k=K, partners=1))
    g = _sim(sc, obs_road=obs_road).host_outputs()
    o = oracle_for(sc, g["state"], g["flags"], g["t"], oracle_mod).obs()
    compare_obs(g, o, K)
    assert (g["road_idx"][0] >= 0).all()


@pytest.mark.parametrize("bins", [64, 256, 1024])
@pytest.mark.parametrize("mates", [1, 2, 4, 5, 9])
def test_ties_in_small_bins(gpu, oracle_mod, mates, bins):
    """Groups of `mates` equal points, so that bins hold 1, 4, 5, ... points and a tie is found
    among the first four or beyond them."""
    rng = np.random.default_rng(mates)
    at = rng.uniform(-30.0, 30.0, (120 // mates, 2))
    pts = rng.permutation(np.repeat(at, mates, axis=0))
    road = [(x, y, -0.4, 0 | 256) for x, y in pts]
    sc = tiny_world([(0.5, -0.25, 1.3, 4.5, 2.0)], extra_road=road, params=_params(top_k=64, partners=1))
    g = _sim(sc, obs_bins=bins).host_outputs()
    o = oracle_for(sc, g["state"], g["flags"], g["t"], oracle_mod).obs()
    compare_obs(g, o, 64)

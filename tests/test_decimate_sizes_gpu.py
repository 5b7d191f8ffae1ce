"""Decimation at the edges of its kernels' size classes (a wave up to 512 points, a workgroup
up to 3072 with the points in LDS and up to 6144 without, the workspace beyond) and on
polylines whose areas tie or cascade: keep masks bit-exact against the oracle."""
import numpy as np
import pytest

from tests.test_decimate_gpu import _compare

pytestmark = pytest.mark.gpu


def _line(kind, n, rng):
    s = np.arange(n) * 0.1
    if kind == "noisy":
        return s + rng.normal(0, 0.01, n), 0.3 * np.sin(s / 6.0) + rng.normal(0, 0.01, n)
    if kind == "straight":  # every area equal (0)
        return s, 0 * s
    if kind == "zigzag":    # every area equal, each removal raises its neighbours'
        return np.arange(n), np.arange(n) % 2.0
    if kind == "steps":     # quantised: many exact ties, collinear runs, repeated points
        return np.floor(4 * s) / 4, np.floor(8 * np.sin(s)) / 8
    return rng.normal(0, 1, n).cumsum(), rng.normal(0, 1, n).cumsum()  # walk: deep cascades


@pytest.mark.parametrize("kind", ["noisy", "straight", "zigzag", "steps", "walk"])
@pytest.mark.parametrize("lens", [[1, 2, 3, 63, 64, 65, 255, 256, 257, 511, 512], [513, 1023, 1024, 1025, 2048, 3071, 3072],
                                  [3073, 0, 4097, 6143, 6144], [6145, 7]])
def test_size_classes(gpu, oracle_mod, kind, lens):
    rng = np.random.default_rng(len(lens))
    pts = [_line(kind, n, rng) for n in lens]
    x, y = (np.concatenate([np.asarray(p[k], np.float64) for p in pts]).astype(np.float32) for k in (0, 1))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    for min_area in (0.0, -0.0, 1e-3, 0.3):
        _compare(oracle_mod, off, x, y, min_area)

"""Decimation by chunks of a polyline that run ahead of each other, at the edges of its size
classes (a wave up to 512 points, a workgroup up to 4096) and on polylines that make the
chunks wait for each other, cascade through them or take the polyline again: keep masks
bit-exact against the oracle."""
import numpy as np
import pytest

from tests.test_decimate_gpu import _compare

pytestmark = pytest.mark.gpu


def _line(kind, n, rng):
    s = np.arange(n) * 0.1
    if kind == "oblique":   # areas of rounding, most of them ties
        return 1.37 * s + 1000, 0.71 * s - 500
    if kind == "circle":    # nearly equal areas
        return 50 * np.cos(s / 50), 50 * np.sin(s / 50)
    if kind == "points":    # a few integer positions: cascades run through whole chunks
        return rng.integers(0, 4, n), rng.integers(0, 4, n)
    if kind == "steps":     # a walk on integer positions
        return rng.integers(-1, 2, n).cumsum(), rng.integers(-1, 2, n).cumsum()
    return s, np.where(rng.random(n) < 0.12, rng.normal(0, 1, n) * np.exp(2 * rng.normal(0, 1, n)), 0.0)  # spikes


@pytest.mark.parametrize("kind", ["oblique", "circle", "points", "steps", "spikes"])
@pytest.mark.parametrize("lens", [[1, 2, 3, 4, 7, 8, 9, 12, 255, 256, 257, 511, 512], [513, 1023, 1025, 2304, 2561],
                                  [4080, 4095, 4096, 4097]])
def test_chunks(gpu, oracle_mod, kind, lens):
    rng = np.random.default_rng(100 + len(lens))
    pts = [_line(kind, n, rng) for n in lens]
    x, y = (np.concatenate([np.asarray(p[k], np.float64) for p in pts]).astype(np.float32) for k in (0, 1))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    for min_area in (0.0, 1e-4, 0.3, 3.0, 1e9):
        _compare(oracle_mod, off, x, y, min_area)

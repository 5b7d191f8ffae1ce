"""Decimation one removal at a time: polylines that are mostly ties (straight lines, rasters, a
straight half) and short ones, at the edges of its chunks of 64 points, of the rule that
chooses it (128 and 256 points, ties in a quarter and in 9 of 20 places) and of the sizes whose
coordinates are in LDS (512 and 3072 points); coordinates that are not finite; keep masks
bit-exact against the oracle."""
import numpy as np
import pytest

from tests.test_decimate_gpu import _compare

pytestmark = pytest.mark.gpu


def _line(kind, n, rng):
    s = np.arange(n) * 0.1
    if kind == "straight":
        return s, 0 * s
    if kind == "raster":
        return np.floor(4 * s) / 4, np.floor(8 * np.sin(s)) / 8
    if kind == "oblique":  # areas of rounding
        return 1.37 * s + 1000, 0.71 * s - 500
    if kind == "vee":      # two straight halves, the last point first
        return np.abs(s - s[n // 2]), s
    share = {"quarter": 4, "half": 2, "most": 20 / 9}[kind]  # straight, then noisy
    return s, np.where(np.arange(n) < n / share, 0.0, rng.normal(0, 0.01, n))


@pytest.mark.parametrize("kind", ["straight", "raster", "oblique", "vee", "quarter", "half", "most"])
@pytest.mark.parametrize("lens", [[1, 2, 3, 4, 63, 64, 65, 66, 127, 128, 129, 130, 191, 193, 255, 256, 257, 258, 511, 512],
                                  [513, 576, 577, 1024, 3071, 3072, 3073], [4095, 4096]])
def test_ties_and_short_lines(gpu, oracle_mod, kind, lens):
    rng = np.random.default_rng(200 + len(lens))
    pts = [_line(kind, n, rng) for n in lens]
    x, y = (np.concatenate([np.asarray(p[k], np.float64) for p in pts]).astype(np.float32) for k in (0, 1))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    for min_area in (0.0, 1e-4, 0.3, 1e9):
        _compare(oracle_mod, off, x, y, min_area)

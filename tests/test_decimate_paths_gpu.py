"""Decimation on the GPU along each path that the host model names (one at a time by the rule,
chunks at the first and the second attempt, one at a time after both), a wave and a
workgroup per polyline, and with coordinates that are not finite: keep masks bit-exact
against the definition."""
import numpy as np
import pytest

from tests.test_decimate_gpu import _compare, _gpu
from tests.test_decimate_model import KINDS, line, model, polylines

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,min_area", [((129, 512), 3.0), ((129, 512), 0.05), ((513, 1500), 3.0)])
def test_each_path(gpu, lens, min_area):
    for k, kind in enumerate(("half", "noisy", "points", "walk", "steps", "spikes")):
        off, x, y = polylines([kind], lens, 150, [9, k])  # (of which the model's test says they reach every path)
        _, keep, path = model(off, x, y, min_area, k)
        got, _ = _gpu(off, x, y, min_area)
        wrong = [(p, int(path[p])) for p in range(len(path)) if (got[off[p]:off[p + 1]] != keep[off[p]:off[p + 1]]).any()]
        assert not wrong, (kind, wrong[:5])


@pytest.mark.parametrize("n", [3, 64, 100, 129, 200, 512, 513, 1000, 3073, 4096, 4097, 6145])
def test_coordinates_that_are_not_finite(gpu, n):
    """Points whose areas are not numbers are never removed and stop nothing: NaN of either sign and
    any payload, infinities (areas inf - inf) and products beyond the largest float, in x, y
    and both.  (The definition is the host model's: the oracle ends at such a point.)"""
    rng = np.random.default_rng(n)
    odd = np.array([0x7fc00000, 0xffc00000, 0xffffffff, 0x7f800001, 0xff800123, 0x7f800000, 0xff800000, 0x7f7fffff, 0xff7fffff],
                   np.uint32).view(np.float32)
    xs, ys, off = [], [], [0]
    for kind in ("noisy", "walk", "half", "steps", "points"):
        x, y = (np.asarray(v, np.float64).astype(np.float32) for v in line(kind, n, rng))
        for v in (x, y):
            at = rng.integers(0, n, max(1, n // 40))
            v[at] = rng.choice(odd, len(at))
        xs.append(x)
        ys.append(y)
        off.append(off[-1] + n)
    off, x, y = np.array(off, np.int32), np.concatenate(xs), np.concatenate(ys)
    for min_area in (0.05, 3.0, 1e30):
        got, _ = _gpu(off, x, y, min_area)
        _, want, _ = model(off, x, y, min_area)
        assert np.array_equal(got, want), np.flatnonzero(got != want)[:5]


def test_kinds_of_the_model(gpu, oracle_mod):
    off, x, y = polylines(KINDS, (1, 700), 400, 21)
    for min_area in (0.002, 0.6):
        _compare(oracle_mod, off, x, y, min_area)

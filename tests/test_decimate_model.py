"""The decimation by chunks on the host: a model of the kernel's chunks, its simultaneous removals
interleaved at random, against the definition.  Every polyline whose order check passes has
the definition's keep mask, and no two chunks write one point in the same round; the kinds
drawn here reach every path (one at a time by the rule, chunks at the first and second attempt,
one at a time after both)."""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
KINDS = ("noisy", "circle", "points", "steps", "spikes", "walk", "raster", "half", "smooth", "zigzag")


def line(kind, n, rng):
    s = np.arange(n) * 0.1
    if kind == "circle":
        return 50 * np.cos(s / 50), 50 * np.sin(s / 50)
    if kind == "points":   # a few integer positions: cascades run through whole chunks
        return rng.integers(0, 6, n), rng.integers(0, 6, n)
    if kind == "steps":    # a walk on integer positions
        return rng.integers(-2, 3, n).cumsum(), rng.integers(-2, 3, n).cumsum()
    if kind == "spikes":
        return s, np.where(rng.random(n) < 0.12, rng.normal(0, 1, n) * np.exp(2 * rng.normal(0, 1, n)), 0.01 * rng.random(n))
    if kind == "walk":
        return rng.normal(0, 0.2, n).cumsum(), rng.normal(0, 0.2, n).cumsum()
    if kind == "raster":
        return np.round(s, 1) + 0.05 * rng.integers(0, 2, n), np.round(np.sin(s / 6) + 0.05 * rng.random(n), 1)
    if kind == "half":
        return s, np.where(np.arange(n) < n // 2, 0.0, rng.normal(0, 0.01, n))
    if kind == "smooth":
        return s, 0.3 * np.sin(s / 6)
    if kind == "zigzag":
        return np.arange(n), np.arange(n) % 2.0 + 1e-3 * rng.integers(0, 3, n)
    return s + rng.normal(0, 0.01, n), 0.3 * np.sin(s / 6) + rng.normal(0, 0.01, n)


def polylines(kinds, lens, count, seed):
    """(offsets, x, y) of `count` polylines of random kinds, with lens[0] to lens[1] points."""
    rng = np.random.default_rng(seed)
    pts = [line(kinds[rng.integers(len(kinds))], int(rng.integers(lens[0], lens[1] + 1)), rng) for _ in range(count)]
    x, y = (np.concatenate([np.asarray(p[k], np.float64) for p in pts]).astype(np.float32) for k in (0, 1))
    return np.concatenate([[0], np.cumsum([len(p[0]) for p in pts])]).astype(np.int32), x, y


_lib = None


def model(off, x, y, min_area, seed=0):
    """(polylines that differ, keep masks of the definition, path of each polyline)."""
    global _lib
    if _lib is None:
        out = os.path.join(tempfile.mkdtemp(), "model.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-o", out,
                               os.path.join(HERE, "decimate_model.cpp")])
        _lib = C.CDLL(out)
        p = C.c_void_p
        _lib.decimate_model.argtypes = [p, C.c_int, p, p, C.c_float, C.c_uint, p, p]
    keep, path = np.zeros(len(x), np.uint8), np.zeros(len(off) - 1, np.int32)
    bad = _lib.decimate_model(off.ctypes.data, len(off) - 1, x.ctypes.data, y.ctypes.data, min_area, seed,
                              keep.ctypes.data, path.ctypes.data)
    return bad, keep, path


@pytest.mark.parametrize("kind", KINDS)
def test_chunks_that_pass_keep_the_definition(kind):
    for k, min_area in enumerate((0.002, 0.05, 0.6, 3.0)):
        bad, _, path = model(*polylines([kind], (129, 420), 400, [k, KINDS.index(kind)]), min_area, k)
        assert bad == 0


def test_longer_polylines():
    bad, _, _ = model(*polylines(KINDS, (513, 2600), 60, 5), 0.05, 1)
    assert bad == 0


def test_definition_is_the_oracles(oracle_mod):
    off, x, y = polylines(KINDS, (1, 300), 200, 7)
    for min_area in (0.0, 0.05, 3.0):
        _, keep, _ = model(off, x, y, min_area)
        assert np.array_equal(keep, oracle_mod.decimate(off, x, y, min_area)[0])


def test_every_path_is_reached():
    seen = set()
    for k, kind in enumerate(("half", "noisy", "points", "walk", "steps", "spikes")):
        for lens in ((129, 512), (513, 1500)):
            seen |= set(model(*polylines([kind], lens, 150, [9, k]), 3.0, k)[2])
    assert seen == {0, 1, 2, 3}

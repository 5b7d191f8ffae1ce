"""Decimation of more polylines than a grid of one workgroup each can hold (2^32 threads: 2^24
workgroups of 256 threads), nearly all of them empty: the few that hold points, at the start
and beyond that number, give the oracle's keep masks."""
import numpy as np
import pytest

from tests.test_decimate_gpu import _compare

pytestmark = pytest.mark.gpu


def test_more_polylines_than_workgroups_fit(gpu, oracle_mod):
    n_poly = (1 << 24) + 3
    at = {0: 20, 1 << 20: 700, (1 << 20) + 1: 40, n_poly - 2: 600, n_poly - 1: 65}
    lens = np.zeros(n_poly, np.int64)
    for k, n in at.items():
        lens[k] = n
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rng = np.random.default_rng(4)
    s = np.arange(off[-1]) * 0.1
    x = (s + rng.normal(0, 0.01, len(s))).astype(np.float32)
    y = (0.3 * np.sin(s / 6) + rng.normal(0, 0.01, len(s))).astype(np.float32)
    kept = _compare(oracle_mod, off, x, y, 0.05)
    assert 0 < kept < len(s)


def test_long_polylines_of_one_workgroup(gpu, oracle_mod):
    """Polylines beyond the LDS sizes at a distance of 512, which one workgroup takes in turn."""
    lens = np.full(1100, 3)
    lens[[3, 515, 1027, 1028]] = [6200, 6145, 6400, 6144]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rng = np.random.default_rng(9)
    s = np.arange(off[-1]) * 0.1
    x = (s + rng.normal(0, 0.01, len(s))).astype(np.float32)
    y = (0.3 * np.sin(s / 6) + rng.normal(0, 0.01, len(s))).astype(np.float32)
    _compare(oracle_mod, off, x, y, 0.05)

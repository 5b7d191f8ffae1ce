"""LIDAR of an agent whose centre lies exactly on a point of a road edge: the two segments that meet
there touch every ray at distance 0 and nowhere else, and hits lie in (0, range], so the agent
sees what it sees without them."""
import dataclasses
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,fov", [(1, 0.0), (2, 0.0), (7, 0.0), (30, 0.0), (200, 0.0), (30, 1.5), (64, 2 * math.pi)])
def test_segments_at_the_agent_are_not_hit(gpu, N, fov):
    from paper_2408_01584_amd import gd as G
    from paper_2408_01584_amd.scenes import Scene, SimParams
    from paper_2408_01584_amd.sim import Sim
    rng = np.random.default_rng(N)
    W = 200
    at = rng.integers(-900, 900, (W, 2)).astype(np.float32)
    # a polyline of three integer points whose middle one is the agent, and others around it
    ends = rng.integers(-30, 31, (W, 2, 2)).astype(np.float32)
    ends[(ends == 0).all(2)] = 7.0
    around = rng.uniform(5, 40, (W, 12, 1)) * np.stack([np.cos(a := rng.uniform(0, 6.28, (W, 12))), np.sin(a)], 2)
    pts = np.concatenate([at[:, None] + np.stack([ends[:, 0], 0 * at, ends[:, 1]], 1), at[:, None] + around], 1).astype(np.float32)
    last = np.zeros((W, 15), np.int32)
    last[:, 2] = last[:, 4::2] = G.GD_META_LAST  # then six segments of two points
    out = []
    for kind in (G.GD_ROAD_EDGE, G.GD_ROAD_LANE):
        meta = last + G.GD_ROAD_EDGE
        meta[:, :3] = last[:, :3] + kind
        f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
        yaw = f(np.where(np.arange(W) % 4 == 0, 0.0, rng.uniform(-math.pi, math.pi, W) if not out else out[0][2]))
        sc = Scene(cfg=0, params=SimParams(top_k=4, partners=0, lidar_rays=N, lidar_fov=float(np.float32(fov))),
                   agent_off=np.arange(W + 1, dtype=np.int32), road_off=(15 * np.arange(W + 1)).astype(np.int32),
                   x=f(at[:, 0]), y=f(at[:, 1]), yaw=yaw, speed=f(np.zeros(W)), length=f(np.full(W, 4.5)),
                   width=f(np.full(W, 2.0)), goal_x=f(at[:, 0] + 50), goal_y=f(at[:, 1]), road_x=f(pts[..., 0].ravel()),
                   road_y=f(pts[..., 1].ravel()), road_dir=f(np.zeros(15 * W)), road_meta=meta.ravel())
        g = Sim(sc).host_outputs()
        out.append((g["lidar"], g["lidar_hit"], yaw))
    (d1, h1, _), (d0, h0, _) = out
    assert N < 7 or (h0 == 1).any()
    assert np.array_equal(h1, h0) and d1.tobytes() == d0.tobytes()

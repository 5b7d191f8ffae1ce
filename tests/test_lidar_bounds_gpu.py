"""LIDAR runs of rays with bounds on what is compared: nearly every ray is outside the oracle's band
and does not graze a short segment, the compared rays hit road edges and agents in the shares
the oracle gives, and their distances differ by at most 1e-5 and what a 1e-4 m move changes,
itself at most 1 cm."""
import dataclasses
import math

import numpy as np
import pytest

from tests._parity import oracle_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,fov", [(30, 0.0), (1024, 0.0), (7, 2 * math.pi), (333, 6.2), (500, 1.0)])
def test_nearly_every_ray_is_compared(gpu, oracle_mod, N, fov):
    from paper_2408_01584_amd import scenes as S
    from paper_2408_01584_amd.sim import Sim
    spec = S.CONFIGS[3]
    parts = [S.make_world(3, w, spec.worlds, dict(spacing=0.2, wobble=0.3, wavelength=40.0, jitter=0.02)) for w in range(3)]
    for p, n in zip(parts, (17, 1, 9)):
        for k in ("x", "y", "yaw", "speed", "length", "width", "goal_x", "goal_y"):
            p[k] = p[k][:n]
    sc = S.assemble(3, parts, dataclasses.replace(spec.params, top_k=8, partners=16, lidar_rays=N,
                                                  lidar_fov=float(np.float32(fov))))
    g = Sim(sc).host_outputs()

    def oracle_at(dx, dy):
        st = np.array(g["state"], np.float64)
        st[0] += dx
        st[1] += dy
        return oracle_for(sc, st, g["flags"], g["t"], oracle_mod, sc.params).obs()
    o = oracle_at(0.0, 0.0)
    off = sum(np.abs(oracle_at(dx, dy)["lidar"] - o["lidar"]) for dx, dy in ((1e-4, 0.0), (0.0, 1e-4)))
    ok = (o["lidar_band"] == 0) & (off <= 0.01)
    assert ok.mean() >= 0.97, ok.mean()
    assert (o["lidar_hit"][ok] == 1).mean() >= 0.4 and (o["lidar_hit"][ok] == 2).any()
    assert np.array_equal(g["lidar_hit"][ok], o["lidar_hit"][ok])
    assert (np.abs(g["lidar"] - o["lidar"]) <= 1e-5 * np.maximum(o["lidar"], 1.0) + off)[ok].all()

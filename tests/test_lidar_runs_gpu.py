"""LIDAR at the edges of its kernel: the fewest and the most rays, runs of rays that wrap past
ray 0 or past +-pi, more candidates with a ray than the list of a wave holds (road edges
every 0.2 m), worlds spread over several workgroups with agent counts that leave waves idle;
hits and distances against the oracle."""
import dataclasses
import math

import numpy as np
import pytest

from tests._parity import oracle_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,fov,dense", [(1, 0.0, False), (2, 0.0, False), (3, 0.0, True), (1024, 0.0, True), (7, 2 * math.pi, True),
                                         (333, 6.2, True), (500, 1.0, True)])
def test_rays_and_cones(gpu, oracle_mod, N, fov, dense):
    from paper_2408_01584_amd import scenes as S
    from paper_2408_01584_amd.sim import Sim
    spec = S.CONFIGS[3]
    parts = [S.make_world(3, w, spec.worlds, dict(spacing=0.2, wobble=0.3, wavelength=40.0, jitter=0.02) if dense else None)
             for w in range(3)]
    for p, n in zip(parts, (17, 1, 9)):
        for k in ("x", "y", "yaw", "speed", "length", "width", "goal_x", "goal_y"):
            p[k] = p[k][:n]
    sc = S.assemble(3, parts, dataclasses.replace(spec.params, top_k=8, partners=16, lidar_rays=N,
                                                  lidar_fov=float(np.float32(fov))))
    sim = Sim(sc)
    g = sim.host_outputs()

    def oracle_at(dx, dy):
        st = np.array(g["state"], np.float64)
        st[0] += dx
        st[1] += dy
        return oracle_for(sc, st, g["flags"], g["t"], oracle_mod, sim.params).obs()
    o = oracle_at(0.0, 0.0)
    ok = o["lidar_band"] == 0
    assert np.array_equal(g["lidar_hit"][ok], o["lidar_hit"][ok])
    # distances: the suite's 1e-5, and what moving the agent by the suite's 1e-4 m band changes
    # (a ray that grazes a short segment turns a rounded coordinate into much more than that)
    off = sum(np.abs(oracle_at(dx, dy)["lidar"] - o["lidar"]) for dx, dy in ((1e-4, 0.0), (0.0, 1e-4)))
    err = np.abs(g["lidar"] - o["lidar"])
    assert (err <= 1e-5 * np.maximum(o["lidar"], 1.0) + off)[ok].all()
    # (two rays look along the road)
    assert (g["lidar_hit"] == 1).any() or N <= 2

"""The launch shape that the library picks by itself, over batch sizes, agents per world, K and
road sizes (few worlds, more than the compute units hold, uneven, no road observation, the
largest K, a world as large as the LDS allows): every output has the bits of a fixed shape."""
import dataclasses

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _scene(counts, road, K):
    from paper_2408_01584_amd import scenes as S
    spec = S.CONFIGS[2]
    parts = []
    for k, n in enumerate(counts):
        p = S.make_world(2, k % 7, spec.worlds)
        for key in ("x", "y", "yaw", "speed", "length", "width", "goal_x", "goal_y"):
            p[key] = np.tile(p[key], -(-n // len(p[key])) if n else 1)[:n]
        p["x"] = p["x"] + 0.11 * np.arange(n)
        for key in ("road_x", "road_y", "road_dir", "road_meta"):
            p[key] = p[key][:road]
        parts.append(p)
    return S.assemble(2, parts, dataclasses.replace(spec.params, top_k=K))


@pytest.mark.parametrize("counts,road,K", [([1], 500, 64), ([3, 0, 5], 800, 0), ([40] * 9, 10000, 960), ([8] * 600, 300, 32),
                                           ([1024], 900, 200), (list(range(1, 120, 7)) * 20, 2000, 100)])
def test_default_shape_changes_no_bit(gpu, counts, road, K):
    from paper_2408_01584_amd import gd as G
    from paper_2408_01584_amd.scenes import make_actions
    from paper_2408_01584_amd.sim import Sim
    sc = _scene(counts, road, K)
    acts = torch.as_tensor(make_actions(2, 2, sc.num_agents), device="cuda")
    outs = []
    fixed = dict(obs_waves=4, obs_bins=64, obs_cands=128, obs_road=G.GD_ROAD_GLOBAL)
    for shape in ({}, fixed):
        sim = Sim(sc, tuned=False, **shape)
        for a in acts:
            sim.step(a)
        outs.append(sim.host_outputs())
        sim.close()
    for k, v in outs[0].items():
        assert v.tobytes() == outs[1][k].tobytes(), k

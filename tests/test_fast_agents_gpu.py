"""Agents at speed on a dense map: more points come within their search radius than the candidate
list holds when it is short, and the grid is scanned again.  The default shape, the shortest
list and the longest give the same bits."""
import dataclasses

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("speed,K", [(30.0, 100), (30.0, 200), (15.0, 64)])
def test_fast_agents_change_no_bit(gpu, speed, K):
    from paper_2408_01584_amd import scenes as S
    from paper_2408_01584_amd.sim import Sim
    sc = S.make_scene(1, worlds=5, dense=dict(spacing=0.4, wobble=0.3, wavelength=40.0, jitter=0.002))
    sc = dataclasses.replace(sc, speed=np.full_like(sc.speed, speed), goal_x=sc.goal_x + np.float32(3000.0),
                             params=dataclasses.replace(sc.params, top_k=K))
    acts = torch.as_tensor(S.make_actions(1, 6, sc.num_agents), device="cuda") * torch.tensor([0.0, 0.05], device="cuda")
    outs = []
    for shape in ({}, dict(obs_cands=128), dict(obs_cands=1024, obs_waves=8)):
        sim = Sim(sc, tuned=False, **shape)
        for a in acts:
            sim.step(a)
        outs.append(sim.host_outputs())
        sim.close()
    assert np.abs(outs[0]["state"][3]).max() > 0.9 * speed
    for o in outs[1:]:
        for k, v in outs[0].items():
            assert v.tobytes() == o[k].tobytes(), k

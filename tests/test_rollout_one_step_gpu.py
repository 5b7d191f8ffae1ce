"""Rollouts of one step, which have kernels of their own (the nearest road edge found without a
list): rewards and gradients against the FP64 oracle, and on a large batch, where shared end
points of segments make exact ties, rewards against the first step of a rollout of two, with
the tolerances of the other rollout tests."""
import dataclasses

import numpy as np
import pytest
import torch

from tests.test_rollout_blocks_gpu import _check, _scene

pytestmark = pytest.mark.gpu

DENSE = dict(spacing=0.2, wobble=0.3, wavelength=40.0, jitter=0.02)


def _actions(sc, T, delta):
    from paper_2408_01584_amd import scenes as S
    return (S.make_delta_actions if delta else S.make_actions)(3, T, sc.num_agents)


@pytest.mark.parametrize("delta,dense,C", [(False, False, 10), (True, False, 1), (True, True, 32), (False, True, 3)])
def test_against_oracle(gpu, oracle_mod, delta, dense, C):
    sc = _scene(delta, worlds=3, **(dict(dense=DENSE) if dense else {}))
    _check(sc, _actions(sc, 1, delta), C, oracle_mod, 0.5 if dense else 0.9)


@pytest.mark.parametrize("delta,away", [(False, 0.0), (True, 0.0), (False, 70.0), (True, 5000.0)])
def test_first_of_two_steps(gpu, delta, away):
    from paper_2408_01584_amd.sim import Sim
    sc = _scene(delta)
    sc = dataclasses.replace(sc, x=sc.x + np.float32(away), goal_x=sc.goal_x + np.float32(away))
    u = torch.as_tensor(_actions(sc, 2, delta), device="cuda")
    sim = Sim(sc)
    (r1, c1, s1, _), (r2, c2, s2, _) = (sim.rollout_fwd(u[:T].contiguous(), 10, obs=True) for T in (1, 2))
    assert torch.equal(c1, c2) and torch.equal(s1[0], s2[0])
    # (another segment of a tie, on the agent's other side, changes a reward by far more)
    assert ((r1[0] - r2[0]).abs() <= 1e-4 * r2[0].abs().clamp_min(1.0)).all()

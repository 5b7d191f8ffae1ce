"""The rollout's observation kernels where a workgroup takes a share of a world's agents (few
worlds and steps) and where it takes all of them (1024 worlds times steps or more): the
observation has the same bits, and the gradient passes the one-step test against 64 bits in
large worlds and in batches of many."""
import dataclasses

import numpy as np
import pytest
import torch

from tests import test_rollout_obs_sizes_gpu as sizes

pytestmark = pytest.mark.gpu


def _repeat(sc, many):
    """many copies of the worlds of sc."""
    arrays = {k: np.tile(getattr(sc, k), many) for k in ("x", "y", "yaw", "speed", "length", "width", "goal_x", "goal_y",
                                                         "road_x", "road_y", "road_dir", "road_meta")}
    offs = {k: np.concatenate([[0], np.cumsum(np.tile(np.diff(getattr(sc, k)), many))]).astype(np.int32)
            for k in ("agent_off", "road_off")}
    return dataclasses.replace(sc, **arrays, **offs)


def _observation(sc, T):
    from paper_2408_01584_amd import scenes as S
    from paper_2408_01584_amd.sim import Sim
    acts = np.tile(S.make_actions(2, T, sc.num_agents // sc.num_worlds), (1, sc.num_worlds, 1))
    return Sim(sc).rollout_fwd(torch.as_tensor(acts, device="cuda"), 8, obs=True)[3]


@pytest.mark.parametrize("n,P,many,T", [(1, 3, 1030, 1), (15, 14, 260, 4), (16, 15, 520, 2), (17, 8, 520, 2), (64, 63, 130, 8),
                                        (65, 64, 130, 8), (130, 129, 70, 15)])
def test_observation_bits(gpu, n, P, many, T):
    one = sizes._scene([n], P)
    lot = _repeat(one, many)
    got = _observation(lot, T).view(T, many, n, -1)
    want = _observation(one, T)
    for w in (0, many // 2, many - 1):
        assert torch.equal(got[:, w], want)


@pytest.mark.parametrize("counts,P,many", [([3, 40], 39, 515), ([1024], 1023, 1), ([1000, 1, 17], 40, 1)])
def test_gradient(gpu, monkeypatch, counts, P, many):
    scene = _repeat(sizes._scene(counts, P), many)
    monkeypatch.setattr(sizes, "_scene", lambda *_: scene)
    sizes.test_one_step_observation_and_gradient(gpu, counts, P)

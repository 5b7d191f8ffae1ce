"""The rollout's observation and its gradient over world sizes and slot counts: fewer lanes
than a wave per observer, several column blocks, slots missing or beyond the world's agents,
and rollouts whose observation gradient is taken in parts (more than 128 steps).  Reference:
the observation formula in plain torch, in 64 bits, its masks taken from the logged
binary32 states (so no agent has to be left out)."""
import dataclasses

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _scene(counts, P):
    from paper_2408_01584_amd import scenes as S
    spec = S.CONFIGS[2]
    parts = []
    for k, n in enumerate(counts):
        w = next(w for w in range(17 * k, 10 ** 6) if len(S.make_world(2, w, spec.worlds)["x"]) >= min(n, 120))
        p = S.make_world(2, w, spec.worlds)
        rep = -(-n // len(p["x"])) if n else 1
        for key in ("x", "y", "yaw", "speed", "length", "width", "goal_x", "goal_y"):
            p[key] = np.tile(p[key], rep)[:n]
        p["x"] = p["x"] + 0.37 * (np.arange(n) // 100)  # (repeated agents moved apart)
        parts.append(p)
    return S.assemble(2, parts, dataclasses.replace(spec.params, partners=P))


def _observe(sc, st, mask_of):
    """obs [A, 3 + 4P] of states st [4, A] (float64, differentiable)."""
    P, rows = sc.params.partners, []
    x, y, th, v = st
    gx, gy = (torch.as_tensor(g, dtype=torch.float64) for g in (sc.goal_x, sc.goal_y))
    for w in range(sc.num_worlds):
        a0, a1 = int(sc.agent_off[w]), int(sc.agent_off[w + 1])
        n = a1 - a0
        if not n:
            continue
        X, Y, TH, V = (q[a0:a1] for q in (x, y, th, v))
        c, s = torch.cos(TH), torch.sin(TH)
        dx, dy = gx[a0:a1] - X, gy[a0:a1] - Y
        ego = torch.stack([V, c * dx + s * dy, -s * dx + c * dy], 1)
        i, sl = torch.arange(n)[:, None], torch.arange(P)[None]
        j = torch.where(sl < i, sl, sl + 1)
        jj = j.clamp(max=n - 1)
        m = (j < n) & mask_of(a0, a1)[torch.arange(n)[:, None], jj]
        dx, dy = X[jj] - X[:, None], Y[jj] - Y[:, None]
        h = torch.remainder(TH[jj] - TH[:, None] + np.pi, 2 * np.pi) - np.pi
        f = torch.stack([c[:, None] * dx + s[:, None] * dy, -s[:, None] * dx + c[:, None] * dy, h, V[jj]], 2)
        rows.append(torch.cat([ego, (f * m[..., None]).flatten(1)], 1))
    return torch.cat(rows)


@pytest.mark.parametrize("counts,P", [([1, 2, 0, 1], 3), ([9, 8, 7], 8), ([17, 30], 12), ([33, 5], 70), ([100, 64, 65], 99),
                                      ([200, 3], 150)])
def test_one_step_observation_and_gradient(gpu, counts, P):
    from paper_2408_01584_amd import scenes as S
    from paper_2408_01584_amd.sim import Sim
    sc = _scene(counts, P)
    A = sc.num_agents
    acts = S.make_actions(2, 1, A)
    go = np.random.default_rng(A).normal(0, 1, (1, A, 3 + 4 * P)).astype(np.float32)
    sim = Sim(sc)
    a_t = torch.as_tensor(acts, device="cuda")
    rew, ck, st, obs = sim.rollout_fwd(a_t, 4, obs=True)
    ga, g0 = sim.rollout_bwd(a_t, ck, torch.zeros_like(rew), 4, want_state0=True,
                             grad_obs=torch.as_tensor(go, device="cuda"), states=st)
    log = st.cpu().numpy()[0]
    R2 = np.float32(sc.params.obs_radius) ** 2

    def mask_of(a0, a1):
        dx, dy = (q[None, a0:a1] - q[a0:a1, None] for q in (log[0], log[1]))
        return torch.as_tensor(dx * dx + dy * dy <= R2)
    # the observation itself, from the logged states
    want = _observe(sc, torch.as_tensor(log).double(), mask_of).numpy()
    got = obs.cpu().numpy()[0]
    off = np.abs(got - want)
    turn = np.zeros(got.shape[1], bool)
    turn[5::4] = True
    off[:, turn] = np.minimum(off[:, turn], np.abs(off[:, turn] - 2 * np.pi))  # (headings at +-pi)
    assert off.max() < 1e-4, off.max()  # coordinates of a few hundred metres, rounded to 32 bits
    # the gradient, through one step of the bicycle model
    s0 = torch.as_tensor(np.stack([sc.x, sc.y, sc.yaw, sc.speed])).double().requires_grad_(True)
    u = torch.as_tensor(acts[0]).double().requires_grad_(True)
    x, y, th, v = s0
    p, L = sc.params, torch.as_tensor(sc.length).double()
    vb = torch.clamp(v + 0.5 * u[:, 0] * p.dt, -p.v_max, p.v_max)
    ts = torch.tan(u[:, 1])
    beta = torch.atan(0.5 * ts)
    st1 = torch.stack([x + vb * torch.cos(th + beta) * p.dt, y + vb * torch.sin(th + beta) * p.dt,
                       th + vb * torch.cos(beta) * ts / L * p.dt, torch.clamp(v + u[:, 0] * p.dt, -p.v_max, p.v_max)])
    loss = (_observe(sc, st1, mask_of) * torch.as_tensor(go[0]).double()).sum()
    w0, wu = torch.autograd.grad(loss, (s0, u))
    for name, g, o in (("state", g0.cpu().numpy(), w0.numpy()), ("action", ga.cpu().numpy()[0].T, wu.numpy().T)):
        err = np.abs(g - o).max(1) / np.sqrt((o ** 2).mean(1))
        assert err.max() < 1e-4, (name, err)


@pytest.mark.parametrize("T,C", [(129, 10), (150, 32)])
def test_gradient_in_parts_matches_oracle_vjp(gpu, oracle_mod, T, C):
    from paper_2408_01584_amd import scenes as S
    from paper_2408_01584_amd.sim import Sim
    from tests.test_rollout_blocks_gpu import _tied
    from tests.test_rollout_obs_gpu import _near_radius_worlds
    sc = _scene([2, 3, 1, 2, 2], 2)
    A = sc.num_agents
    acts = 0.3 * S.make_actions(2, T, A)
    rng = np.random.default_rng(T)
    gr = rng.uniform(0.5, 1.5, (T, A)).astype(np.float32)
    go = rng.normal(0, 1, (T, A, 11)).astype(np.float32)
    sim = Sim(sc)
    a_t = torch.as_tensor(acts, device="cuda")
    _, ck, st, _ = sim.rollout_fwd(a_t, C, obs=True)
    ga, _ = sim.rollout_bwd(a_t, ck, torch.as_tensor(gr, device="cuda"), C, grad_obs=torch.as_tensor(go, device="cuda"),
                            states=st)
    ga = ga.cpu().numpy()
    orc = oracle_mod.OracleSim(sc)
    ref = orc.rollout(acts.astype(np.float64), tol=1e-3)
    oga, _ = orc.rollout_vjp(acts.astype(np.float64), gr.astype(np.float64), go.astype(np.float64))
    world = np.repeat(np.arange(sc.num_worlds), np.diff(sc.agent_off))
    bad = _near_radius_worlds(sc, ref["states"], sc.params.obs_radius)
    np.logical_or.at(bad, world, (ref["unstable"] != 0) | _tied(sc, ref["states"]))
    ok = ~bad[world]
    assert ok.sum() >= 4, bad
    d = (ga - oga)[:, ok].transpose(1, 0, 2).reshape(ok.sum(), -1)
    den = np.linalg.norm(oga[:, ok].transpose(1, 0, 2).reshape(ok.sum(), -1), axis=1)
    assert (np.linalg.norm(d, axis=1) / den).max() < 1e-3

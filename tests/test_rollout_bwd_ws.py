"""The rollout backward keeps nothing in the simulator: the handle's workspace does not depend on
the partner slots, and gd_rollout_bwd_ws checks the workspace of the call (no GPU needed)."""
import numpy as np

from tests.test_abi import G, _cfg  # noqa: F401  (G: fixture)


def test_handle_workspace_holds_no_rollout_scratch(G):  # noqa: F811
    ao, ro = np.array([0, 64, 100], np.int32), np.array([0, 100, 150], np.int32)
    sizes = {G.gd_workspace_size(_cfg(G, partners=p), ao, ro) for p in (-1, 0, 3, 63)}
    assert len(sizes) == 1, sizes


def test_null_handles(G):  # noqa: F811
    L = G.lib()
    assert L.gd_rollout_bwd_ws(None, None, None, 1, 1, None, None, None, None, None, None, 0, None) == G.GD_E_ARG
    assert L.gd_rollout_bwd_workspace_size(None, 1, None) == G.GD_E_ARG

"""GPU checks of the default configuration on small layouts, where the library
gives a drone four or eight lanes: bitwise the results of the one-lane
configuration that it reports, at the environment sizes where a group of lanes
or a round of candidates ends, idle lanes and tiny environments included, with
and without observations, on layered flight and on a dense coplanar grid, and
through a captured rollout."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import md, workloads as wl
from test_gpu_block_sweep import _mixed

pytestmark = pytest.mark.gpu


def _rpm(w, steps, seed):
    n = w["action"].shape[2]
    u = np.random.default_rng(seed).uniform(-0.1, 0.1, (steps, 4, n))
    w = dict(w, act_type="rpm", action_per_step=True)
    w["action"] = (pu.hover_rpm() * (1 + u)).astype(np.float32)
    return w


LAYOUTS = {
    "eight_lanes": lambda: _mixed([2, 24, 1, 32, 31, 33, 3, 0, 17, 16, 15, 40, 8, 7, 9], 21),
    "eight_lanes_112": lambda: _mixed([112, 5, 111, 64, 65, 1, 97], 22),
    "four_lanes_small": lambda: _mixed([2, 4, 5, 8, 23, 1, 7, 16, 17, 9, 0, 12] * 9, 23),
    "four_lanes": lambda: wl.thin_envs(wl.lattice(n_envs=900, shape=(4, 4, 2), seed=24), 25),
    "dense_grid": lambda: wl.ragged_grid(pu.hover_rpm(), n_envs=200, n_steps=20, seed=26),
    "rpm": lambda: _rpm(_mixed([32, 30, 2, 64, 11], 27), 20, 28),
}


@pytest.mark.parametrize("obs", [0, 1, 12])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_default_equals_one_lane(name, obs):
    w = LAYOUTS[name]()
    waves = 1
    while 64 * waves < int(np.diff(w["env_offsets"]).max()):
        waves *= 2
    got = []
    for cfg in (None, dict(lanes_per_drone=1, unroll=4, waves_per_group=waves, pair_symmetric=0)):
        print("%s obs %d %s" % (name, obs, cfg), flush=True)
        g = pu.DeviceRun(w, cfg=cfg)
        assert md.md_get_launch_config(g.ctx)["lanes_per_drone"] == 1
        rows = [g.run(k, obs_slots=obs) for k in (5, 12)]
        got.append((g.snapshot(), rows))
        g.close()
    for k in ("p", "q", "v", "w", "rpm", "pid_int"):
        np.testing.assert_array_equal(got[0][0][k], got[1][0][k], err_msg=k)
    if obs:
        for a, b in zip(got[0][1], got[1][1]):
            np.testing.assert_array_equal(a, b)


def test_captured_rollout_on_the_default_configuration():
    import torch
    w = LAYOUTS["eight_lanes"]()
    g, h = pu.DeviceRun(w), pu.DeviceRun(w)
    try:
        graph = md.md_rollout_graph_create(g.ctx, g.state, g.action, False, steps_per_launch=5, n_launches=2)
        for _ in range(3):
            md.md_graph_launch(graph)
            torch.cuda.synchronize()
            for l in range(2):
                md.md_step(h.ctx, h.state, h.action, False, None, 0, 5, 5 * l)
            a, b = g.snapshot(), h.snapshot()
            for k in ("p", "q", "v", "w", "rpm", "pid_int"):
                np.testing.assert_array_equal(a[k], b[k])
        md.md_graph_destroy(graph)
    finally:
        g.close()
        h.close()

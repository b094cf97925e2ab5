"""GPU checks of the tested sweeps across the end of their tests: swarms that
start drawn together, where the tests are given up for some steps, and fly
apart.  One launch, whose tests come and go, against launches of a single step,
each of which tests at its start: bitwise the same, for every sweep that
tests."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import md, workloads as wl

pytestmark = pytest.mark.gpu

ROT = dict(lanes_per_drone=1, unroll=1, waves_per_group=8, pair_symmetric=3)
ONE = dict(lanes_per_drone=1, unroll=4, waves_per_group=1, pair_symmetric=0)
# environments, lattice, configuration, kind
CASES = {
    "rotation32": (21, (4, 4, 2), ROT, ""), "rotation64": (13, (8, 4, 2), ROT, ""),
    "rotation64_wind": (13, (8, 4, 2), ROT, "wind"), "rotation32_randomized": (13, (4, 4, 2), ROT, "dr"),
    "rk4_rotation32": (21, (4, 4, 2), ROT, "rk4"), "rk4_rotation64": (13, (8, 4, 2), ROT, "rk4"),
    "one_lane_wind": (21, (4, 4, 2), ONE, "wind"), "one_lane_wind64": (9, (8, 4, 2), ONE, "wind"),
    "one_lane_randomized": (21, (4, 4, 2), ONE, "dr"), "one_lane_randomized64": (9, (8, 4, 2), ONE, "dr"),
    "block": (5, (10, 8, 2), None, ""), "block_rk4": (5, (10, 8, 2), None, "rk4"),
    "block_wind": (5, (10, 8, 2), None, "wind"),
}


@pytest.mark.parametrize("obs", [0, 1])
@pytest.mark.parametrize("scale", [0.05, 0.35, 0.6])
@pytest.mark.parametrize("name", list(CASES))
def test_one_launch_equals_single_steps(name, scale, obs):
    n_envs, shape, cfg, kind = CASES[name]
    w = wl.lattice(n_envs=n_envs, shape=shape, n_steps=1, seed=14)
    w["state"]["p"][:2] *= np.float32(scale)
    # every second environment flies outwards, past the tests' limit again
    m = shape[0] * shape[1] * shape[2]
    far = (np.arange(n_envs * m) // m) % 2 == 0
    w["state"]["v"][:2, far] = w["state"]["p"][:2, far] * np.float32(8.0 / scale)
    if kind == "rk4":
        w["integrator"] = "rk4"
    if kind in ("wind", "dr"):
        w["wind"] = wl.dr_wind(w, 3)
    if kind == "dr":
        w["dr"] = wl.domain_randomization(w, 4)
    steps, got = 75, []
    for split in ((steps,), (1,) * steps):
        print("%s scale %g, %d launches" % (name, scale, len(split)), flush=True)
        g = pu.DeviceRun(w, cfg=cfg)
        for k in split:
            row = g.run(k, obs_slots=obs)
        got.append((g.snapshot(), row))
        g.close()
    if obs:
        np.testing.assert_array_equal(got[1][1], got[0][1])
    for k in got[0][0]:
        np.testing.assert_array_equal(got[1][0][k], got[0][0][k], err_msg=k)

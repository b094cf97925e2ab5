"""GPU checks of the rotation sweep's workgroups: a launch of 500 steps that
stores rows and fills the GPU runs in groups of waves, two launches of 250 run
every wave by itself.  Same state and same last row, bit for bit, for Euler at
three environment sizes, wind and Runge-Kutta."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import md, workloads as wl

pytestmark = pytest.mark.gpu

CASES = {"euler16": (16380, (4, 2, 2)), "euler32": (8190, (4, 4, 2)), "euler64": (4095, (8, 4, 2)),
         "wind32": (6500, (4, 4, 2)), "rk4_32": (6500, (4, 4, 2)), "rk4_64": (4095, (8, 4, 2))}


@pytest.mark.parametrize("name", list(CASES))
def test_a_grouped_launch_equals_waves_of_their_own(name):
    n_envs, shape = CASES[name]
    w = wl.lattice(n_envs=n_envs, shape=shape, n_steps=1, seed=12)
    if name.startswith("rk4"):
        w["integrator"] = "rk4"
    if name.startswith("wind"):
        w["wind"] = wl.dr_wind(w, 3)
    got = []
    for split in ((500,), (250, 250)):
        print("%s, launches of %s steps" % (name, split), flush=True)
        g = pu.DeviceRun(w, cfg=dict(lanes_per_drone=1, unroll=1, waves_per_group=16, pair_symmetric=3))
        for k in split:
            row = g.run(k, obs_slots=1)
        got.append((g.snapshot(), row))
        g.close()
    np.testing.assert_array_equal(got[1][1], got[0][1])
    for k in got[0][0]:
        np.testing.assert_array_equal(got[1][0][k], got[0][0][k], err_msg=k)

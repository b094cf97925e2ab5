"""GPU check of the default configuration on small layouts, where the library
gives a drone four or eight lanes: bitwise the results of one lane per drone
(asked for with another unroll than the default's, which is the same sum)."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import md
from test_gpu_lanes import LAYOUTS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("obs", [0, 1, 12])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_default_equals_one_lane_of_another_unroll(name, obs):
    w = LAYOUTS[name]()
    waves = 1
    while 64 * waves < int(np.diff(w["env_offsets"]).max()):
        waves *= 2
    one = dict(lanes_per_drone=1, unroll=2, waves_per_group=waves, pair_symmetric=0)
    got = []
    for cfg in (None, one):
        print("%s obs %d %s" % (name, obs, cfg), flush=True)
        g = pu.DeviceRun(w, cfg=cfg)
        assert (md.md_get_launch_config(g.ctx) == one) == (cfg is not None)
        rows = [g.run(k, obs_slots=obs) for k in (5, 12)]
        got.append((g.snapshot(), rows))
        g.close()
    for k in ("p", "q", "v", "w", "rpm", "pid_int"):
        np.testing.assert_array_equal(got[0][0][k], got[1][0][k], err_msg=k)
    if obs:
        for a, b in zip(got[0][1], got[1][1]):
            np.testing.assert_array_equal(a, b)

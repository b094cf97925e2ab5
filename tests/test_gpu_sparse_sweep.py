"""GPU checks of the sweeps that test every pair before they evaluate any: on
layered lattices, where few pairs pass, on the same lattices drawn together
until most do (the sweeps then skip the tests for some steps), and with
partners exactly above one another and exactly level.  The rotation sweep must
stay bitwise equal to the wave-permute sweep, which evaluates every pair; the
block sweep is held to the oracle step by step."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import md, workloads as wl

pytestmark = pytest.mark.gpu

SHAPES = {16: (4, 2, 2), 32: (4, 4, 2), 64: (8, 4, 2)}


def _packed(n_envs, shape, scale, seed):
    w = wl.lattice(n_envs=n_envs, shape=shape, n_steps=40, seed=seed)
    s = w["state"]
    s["p"][:2] *= np.float32(scale)
    w["action"][:, :2] *= np.float32(scale)
    m = shape[0] * shape[1] * shape[2]
    # in every third environment the columns stand exactly above one another
    # and the layers are exactly level
    p = s["p"].reshape(3, n_envs, m)
    p[0:2, ::3, 1::2] = p[0:2, ::3, 0::2]
    p[2, ::3, 0::2] = np.float32(0.5)
    p[2, ::3, 1::2] = np.float32(1.5)
    return w


@pytest.mark.parametrize("scale", [1.0, 0.4, 0.05])
@pytest.mark.parametrize("kind", ["euler", "rk4", "wind"])
@pytest.mark.parametrize("m", [16, 32, 64])
def test_rotation_sweep_equals_permute_sweep(m, kind, scale):
    w = _packed(37, SHAPES[m], scale, 8)
    if kind == "rk4":
        w["integrator"] = "rk4"
    elif kind == "wind":
        w["wind"] = wl.dr_wind(w, 3)
    got = []
    for sym, waves in ((2, 1), (3, 1), (3, 8)):
        print("m %d %s scale %g sweep %d, %d waves" % (m, kind, scale, sym, waves), flush=True)
        g = pu.DeviceRun(w, cfg=dict(lanes_per_drone=1, unroll=1, waves_per_group=waves, pair_symmetric=sym))
        obs = g.run(21, obs_slots=21)
        got.append((g.snapshot(), obs))
        g.close()
    for s, obs in got[1:]:
        np.testing.assert_array_equal(obs, got[0][1])
        for k in ("p", "q", "v", "w", "rpm", "pid_int"):
            np.testing.assert_array_equal(s[k], got[0][0][k])


@pytest.mark.parametrize("scale", [1.0, 0.4, 0.05])
def test_block_sweep_per_step(scale):
    w = _packed(6, (10, 8, 2), scale, 9)  # 160 drones
    g = pu.DeviceRun(w)
    try:
        for k in (0, 1, 3, 12):
            if k > g.step_index:
                g.run(k - g.step_index)
            s0 = g.snapshot()
            g.run(1)
            ref, _, _ = pu.oracle_one_step(w, s0, k)
            pu.assert_blocks(g.snapshot(), ref, what="scale %g step %d" % (scale, k))
    finally:
        g.close()


@pytest.mark.parametrize("scale", [1.0, 0.4, 0.05])
@pytest.mark.parametrize("kind", ["wind", "randomized"])
@pytest.mark.parametrize("layout", ["uniform32", "ragged64"])
def test_one_lane_sweep_equals_matrix_sweep(layout, kind, scale):
    """The one-lane sweep of the kernels with wind or randomisation against
    the LDS-matrix sweep, which evaluates every pair and sums in the same
    order."""
    if layout == "uniform32":
        w = _packed(23, (4, 4, 2), scale, 10)
    else:
        w = wl.thin_envs(_packed(31, (8, 4, 2), scale, 11), 12, m_lo=1)
    if kind == "wind":
        w["wind"] = wl.dr_wind(w, 3)
    else:
        w = dict(w, dr=wl.domain_randomization(w, 4), wind=wl.dr_wind(w, 5))
    got = []
    for sym in (1, 0):
        print("%s %s scale %g sweep %d" % (layout, kind, scale, sym), flush=True)
        g = pu.DeviceRun(w, cfg=dict(lanes_per_drone=1, unroll=4, waves_per_group=2, pair_symmetric=sym))
        obs = g.run(21, obs_slots=21)
        got.append((g.snapshot(), obs))
        g.close()
    np.testing.assert_array_equal(got[1][1], got[0][1])
    for k in ("p", "q", "v", "w", "rpm", "pid_int", "wind"):
        np.testing.assert_array_equal(got[1][0][k], got[0][0][k])

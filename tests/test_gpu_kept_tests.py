"""GPU checks of the sweeps that keep the outcomes of their pairs' tests until a
drone has moved: one launch of many steps must equal, bit for bit, as many
launches of one step, which form every test anew.  Standing, slow and fast
drones (the outcomes last for the launch, some steps, or less than one), sparse
and dense lattices, environments that end inside a wave."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import workloads as wl

pytestmark = pytest.mark.gpu

STEPS = 48
LAYOUTS = {
    # name: (environments, lattice, thinned, configuration)
    "rotation64": (13, (8, 4, 2), False, dict(waves_per_group=1, pair_symmetric=3)),
    "rotation32": (25, (4, 4, 2), False, dict(waves_per_group=1, pair_symmetric=3)),
    "rotation16": (25, (4, 2, 2), False, dict(waves_per_group=1, pair_symmetric=3)),
    "block128": (5, (8, 8, 2), False, None),
    "block_ragged": (6, (10, 10, 2), True, None),
    "randomized32": (21, (4, 4, 2), False, dict(waves_per_group=1, pair_symmetric=0)),
    "randomized_ragged": (21, (4, 4, 2), True, dict(waves_per_group=1, pair_symmetric=0)),
}
CASES = [(name, kind) for name in sorted(LAYOUTS) for kind in ("euler", "rk4")
         if not (kind == "rk4" and name.startswith("randomized"))]


@pytest.mark.parametrize("speed", [0.0, 0.6, 15.0])
@pytest.mark.parametrize("scale", [1.0, 0.3])
@pytest.mark.parametrize("layout,kind", CASES)
def test_one_launch_equals_single_steps(layout, kind, scale, speed):
    randomized = layout.startswith("randomized")
    n_envs, shape, thinned, cfg = LAYOUTS[layout]
    w = wl.lattice(n_envs=n_envs, shape=shape, n_steps=STEPS, seed=21)
    s = w["state"]
    s["p"][:2] *= np.float32(scale)
    w["action"][:, :2] *= np.float32(scale)
    s["v"][:] += (speed * np.random.default_rng(22).uniform(-1, 1, s["v"].shape)).astype(np.float32)
    if thinned:
        w = wl.thin_envs(w, 23, m_lo=shape[0] * shape[1] + 13 if layout == "block_ragged" else 1)
    if randomized:
        w = dict(w, dr=wl.domain_randomization(w, 4), wind=wl.dr_wind(w, 5))
    if kind == "rk4":
        w["integrator"] = "rk4"
    if cfg is not None:
        cfg = dict(cfg, lanes_per_drone=1, unroll=1 if cfg["pair_symmetric"] else 4)
    got = []
    for chunk in (1, STEPS):
        print("%s %s scale %g speed %g: %d steps a launch" % (layout, kind, scale, speed, chunk), flush=True)
        g = pu.DeviceRun(w, cfg=cfg)
        for _ in range(STEPS // chunk):
            g.run(chunk)
        got.append(g.snapshot())
        g.close()
    # (a randomised drone that starts at 15 m/s leaves the model's range, in
    # the oracle too, and its position becomes a NaN: compared like any value)
    for k in ("p", "q", "v", "w", "rpm", "pid_int"):
        np.testing.assert_array_equal(got[1][k], got[0][k])


@pytest.mark.parametrize("shape", [(2, 1, 1), (1, 2, 2), (2, 2, 2)])
def test_small_runge_kutta_rotation_equals_permute(shape):
    """The rotation by batches where an environment has fewer shifts than a
    batch, or one batch exactly."""
    w = wl.lattice(n_envs=101, shape=shape, n_steps=STEPS, seed=24)
    w["state"]["p"][:2] *= np.float32(0.2)
    w["action"][:, :2] *= np.float32(0.2)
    w["integrator"] = "rk4"
    got = []
    for sym in (2, 3):
        print("%s sweep %d" % (shape, sym), flush=True)
        g = pu.DeviceRun(w, cfg=dict(lanes_per_drone=1, unroll=1, waves_per_group=1, pair_symmetric=sym))
        g.run(STEPS)
        got.append(g.snapshot())
        g.close()
    for k in ("p", "q", "v", "w", "rpm", "pid_int"):
        np.testing.assert_array_equal(got[1][k], got[0][k])


@pytest.mark.parametrize("kind", ["euler", "rk4"])
@pytest.mark.parametrize("n_envs,shape", [(8192, (4, 4, 2)), (16384, (4, 2, 2)), (4096, (8, 4, 2))])
def test_long_launch_equals_short_ones(n_envs, shape, kind):
    """A long launch with rows that fills the chip takes workgroups of several
    waves, and up to 32 drones no tests; its parts take one wave each."""
    w = wl.lattice(n_envs=n_envs, shape=shape, n_steps=750, seed=25)
    if kind == "rk4":
        w["integrator"] = "rk4"
    got = []
    for chunk in (750, 375):
        print("%d x %s %s: %d steps a launch" % (n_envs, shape, kind, chunk), flush=True)
        g = pu.DeviceRun(w, cfg=dict(lanes_per_drone=1, unroll=1, waves_per_group=16, pair_symmetric=3))
        for _ in range(750 // chunk):
            obs = g.run(chunk, obs_slots=3)
        got.append((g.snapshot(), obs))
        g.close()
    np.testing.assert_array_equal(got[1][1], got[0][1])
    for k in ("p", "q", "v", "w", "rpm", "pid_int"):
        np.testing.assert_array_equal(got[1][0][k], got[0][0][k])

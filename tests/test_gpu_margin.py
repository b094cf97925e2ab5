"""GPU checks of the pair tests where the wake's width passes through 0 (C2 dz +
C3 = 0, a height of 0.6875 m): partners that far above and a float32 step or a
few to the side, whose terms the tests may not leave out.  The rotation sweep
against the permute sweep and the one-lane sweep under wind against the
LDS-matrix sweep, both of which evaluate every pair: bitwise."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import md, workloads as wl

pytestmark = pytest.mark.gpu


def _stacked(step, seed):
    """16 sites 20 cm apart, a drone at 0.5 m and one 0.6875 m above it, every
    upper drone the given number of float32 steps to the side; the environments
    differ in the last bits of the height."""
    n_envs = 6
    w = wl.lattice(n_envs=n_envs, shape=(4, 4, 2), n_steps=4, seed=seed)
    p = w["state"]["p"].reshape(3, n_envs, 32)
    x, y = np.meshgrid([0.3, 0.5, 0.7, 0.9], [0.3, 0.5, 0.7, 0.9])
    for e in range(n_envs):
        p[0, e] = np.tile(x.ravel(), 2).astype(np.float32)
        p[1, e] = np.tile(y.ravel(), 2).astype(np.float32)
        p[2, e, :16] = np.float32(0.5)
        top = np.float32(1.1875)
        for _ in range(abs(e - 3) // 2):
            top = np.nextafter(top, np.float32(2.0 if e > 3 else 0.0), dtype=np.float32)
        p[2, e, 16:] = top
        for _ in range(step):
            p[0, e, 16:] = np.nextafter(p[0, e, 16:], np.float32(10.0), dtype=np.float32)
    w["state"]["v"][:] = 0
    return w


def _run(w, sym, waves, steps):
    g = pu.DeviceRun(w, cfg=dict(lanes_per_drone=1, unroll=1, waves_per_group=waves, pair_symmetric=sym))
    try:
        g.run(steps)
        return g.snapshot()
    finally:
        g.close()


@pytest.mark.parametrize("step", [0, 1, 2, 3, 4, 8])
@pytest.mark.parametrize("kind", ["euler", "wind"])
def test_no_needed_pair_is_left_out(kind, step):
    w = _stacked(step, 40 + step)
    if kind == "wind":
        w["wind"] = wl.dr_wind(w, 3)
    for steps in (1, 2):
        print("%s, %d float32 steps to the side, %d time steps" % (kind, step, steps), flush=True)
        ref = _run(w, 2 if kind == "euler" else 1, 1, steps)
        got = _run(w, 3 if kind == "euler" else 0, 1, steps)
        for k in ("p", "q", "v", "w", "rpm", "pid_int"):
            np.testing.assert_array_equal(got[k], ref[k], err_msg=k)


def test_heights_next_to_zero_with_a_bounded_gap():
    """Heights 0 and 1e-21: with dw_dz_min the term stays finite and a partner
    outside the wake adds 0, evaluated or not."""
    w = _stacked(0, 50)
    p = w["state"]["p"].reshape(3, 6, 32)
    p[0, :, 16:] += np.float32(0.1)
    p[2, :, :16] = 0.0
    p[2, :, 16:] = np.float32(1e-21)
    par = pu.params()
    par.dw_dz_min = 0.01
    got = []
    for sym in (2, 3):
        g = pu.DeviceRun(w, p=par, cfg=dict(lanes_per_drone=1, unroll=1, waves_per_group=1, pair_symmetric=sym))
        g.run(2)
        got.append(g.snapshot())
        g.close()
    for k in ("p", "q", "v", "w", "rpm", "pid_int"):
        assert np.isfinite(got[0][k]).all()
        np.testing.assert_array_equal(got[1][k], got[0][k], err_msg=k)

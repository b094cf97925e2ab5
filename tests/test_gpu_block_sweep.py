"""GPU checks of the block-symmetric sweep (environments of more than 112
drones under the one-lane all-pairs configuration): per-step parity with the
oracle at the sizes where waves begin and end, mixed with small environments
that keep the ascending sweep, for every integrator and disturbance that
shares it; bitwise invariance to the workgroup size, the unroll, the
environment order and the other environments of the layout."""
import numpy as np
import pytest

import parity_util as pu
from paper_2606_08039_amd import md, workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [113, 128, 129, 7, 192, 1, 200, 256, 64, 257, 112, 320, 0, 511, 512]
LARGE = [1024, 1000, 577, 3, 130]


def _mixed(sizes, seed):
    """Layered lattices, environment e keeping a random sizes[e] of its drones."""
    n = max(sizes)
    shape = (16, 16, 2) if n <= 512 else (16, 32, 2)
    w = wl.lattice(n_envs=len(sizes), shape=shape, n_steps=20, seed=seed)
    rng = np.random.default_rng(seed + 9)
    m = shape[0] * shape[1] * shape[2]
    idx = np.concatenate([e * m + np.sort(rng.choice(m, k, replace=False)) for e, k in enumerate(sizes)])
    idx = idx.astype(np.int64)
    out = dict(w)
    out["env_offsets"] = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    out["state"] = {k: np.ascontiguousarray(v[:, idx]) for k, v in w["state"].items()}
    out["action"] = np.ascontiguousarray(w["action"][:, :, idx])
    out.pop("lattice_points")
    return out


def _run(w, cfg, steps):
    g = pu.DeviceRun(w, cfg=cfg)
    g.run(steps)
    s = g.snapshot()
    g.close()
    return s


def _cfg(waves, unroll=4):
    return dict(lanes_per_drone=1, unroll=unroll, waves_per_group=waves, pair_symmetric=0)


@pytest.mark.parametrize("kind", ["euler", "rk4", "randomized", "wind", "dz_min", "large"])
def test_per_step_parity(kind):
    w = _mixed(LARGE if kind == "large" else SIZES, 5)
    p = None
    if kind == "rk4":
        w["integrator"] = "rk4"
    elif kind == "randomized":
        w = wl.randomized(w, 11)
    elif kind == "wind":
        w["wind"] = wl.dr_wind(w, 12)
    if kind == "dz_min":
        p = pu.params()
        p.dw_dz_min = 0.05
    g = pu.DeviceRun(w, p=p)
    try:
        for k in (0, 1, 6):
            if k > g.step_index:
                g.run(k - g.step_index)
            s0 = g.snapshot()
            print("%s step %d" % (kind, k), flush=True)
            g.run(1)
            s1 = g.snapshot()
            if kind == "dz_min":
                continue  # the oracle's parameters are the defaults: see the sweeps' comparison below
            ref, _, idx = pu.oracle_one_step(w, s0, k)
            pu.assert_blocks(s1, ref, idx, what="%s step %d" % (kind, k))
        if kind == "dz_min":
            # two lanes per drone: the all-pairs sweep, other summation order
            h = pu.DeviceRun(w, p=p, cfg=dict(lanes_per_drone=2, unroll=1, waves_per_group=16, pair_symmetric=0))
            h.run(7)
            pu.assert_blocks(s1, h.snapshot(), what="two lanes")
            h.close()
    finally:
        g.close()


def test_bitwise_invariance():
    w = _mixed(SIZES, 6)
    ref = _run(w, _cfg(8), 9)
    for cfg in (_cfg(16), _cfg(8, 1), None):
        got = _run(w, cfg, 9)
        for k in ("p", "q", "v", "w"):
            np.testing.assert_array_equal(got[k], ref[k], err_msg="%s %s" % (cfg, k))
    perm = np.random.default_rng(1).permutation(len(SIZES))
    wp = wl.permute_envs(w, perm)
    got = _run(wp, None, 9)
    for k in ("p", "q", "v", "w"):
        np.testing.assert_array_equal(got[k], ref[k][:, wp["drone_index"]])
    # alone in its layout: one large environment, one small one
    for e in (SIZES.index(200), SIZES.index(112), SIZES.index(129)):
        i0, i1 = w["env_offsets"][e], w["env_offsets"][e + 1]
        one = dict(w, env_offsets=np.array([0, i1 - i0], dtype=np.int32),
                   state={k: np.ascontiguousarray(v[:, i0:i1]) for k, v in w["state"].items()},
                   action=np.ascontiguousarray(w["action"][:, :, i0:i1]))
        got = _run(one, None, 9)
        for k in ("p", "q", "v", "w"):
            np.testing.assert_array_equal(got[k], ref[k][:, i0:i1], err_msg="environment of %d" % SIZES[e])

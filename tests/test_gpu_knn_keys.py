"""The neighbour ranking by keys (distance and number in one word) against the
exact one where they could part: environment sizes around 8, 9 and 64, exactly
equal distances (a regular grid), distances equal but for the bits that the
number takes, coincident drones, and positions beyond the keys' range."""
import numpy as np
import pytest

import oracle as orc
import parity_util as pu
from paper_2606_08039_amd import md, workloads as wl

pytestmark = pytest.mark.gpu


def _near_ties(w, seed):
    """Horizontal positions on a circle around each environment's first drone,
    its radius a few float32 steps apart from drone to drone."""
    rng = np.random.default_rng(seed)
    p = w["state"]["p"]
    off = w["env_offsets"]
    for e in range(len(off) - 1):
        m = off[e + 1] - off[e]
        if m < 2:
            continue
        a = rng.permutation(np.arange(1, m)) * (2 * np.pi / m)
        r = 1.0 + rng.integers(0, 60, m - 1) * 2.0 ** -23
        p[0, off[e]:off[e + 1]] = np.concatenate([[0.0], r * np.cos(a)])
        p[1, off[e]:off[e + 1]] = np.concatenate([[0.0], r * np.sin(a)])
    return w


def _far(w):
    w["state"]["p"][0, ::7] += np.float32(3e18)
    w["state"]["p"][1, ::11] = np.float32(np.inf)
    return w


def _together(w):
    p = w["state"]["p"]
    p[:2, 1::2] = p[:2, 0:-1:2][:, :p[:2, 1::2].shape[1]]
    return w


def _thin(shape, n, seed):
    return wl.thin_envs(wl.lattice(n_envs=n, shape=shape, seed=seed), seed + 1, m_lo=1)


CASES = {
    "lattice64": lambda: wl.lattice(n_envs=20, shape=(8, 4, 2), seed=1),
    "sizes": lambda: _thin((4, 4, 2), 80, 2),
    "nine": lambda: wl.lattice(n_envs=40, shape=(3, 3, 1), seed=3),
    "grid": lambda: wl.ragged_grid(pu.hover_rpm(), n_envs=60, n_steps=1, seed=4),
    "near_ties": lambda: _near_ties(_thin((8, 4, 2), 40, 5), 6),
    "together": lambda: _together(wl.lattice(n_envs=30, shape=(4, 4, 2), seed=7)),
    "far": lambda: _far(wl.lattice(n_envs=30, shape=(4, 4, 2), seed=8)),
    "sixty_five": lambda: wl.lattice(n_envs=7, shape=(13, 5, 1), seed=9),
}


@pytest.mark.parametrize("name", list(CASES))
def test_datagen_neighbours(name):
    import torch
    print(name, flush=True)
    w = CASES[name]()
    g = pu.DeviceRun(w)
    X, Y = torch.zeros((g.n, 64), device="cuda"), torch.zeros((g.n, 6), device="cuda")
    nbr = torch.zeros((g.n, 8), dtype=torch.int32, device="cuda")
    md.md_datagen(g.ctx, g.state, 7, X, Y, nbr)
    torch.cuda.synchronize()
    s = pu.to_oracle_state(g.snapshot())
    g.close()
    ref = orc.knn(w["env_offsets"], s["p"], 8)
    # candidates at a non-finite distance, which the oracle ranks last, never
    # enter the library's lists
    xy = s["p"][:2]
    with np.errstate(invalid="ignore"):
        d = xy[:, ref] - xy[:, :, None]
    ref = np.where(np.isfinite(d).all(0), ref, -1)
    np.testing.assert_array_equal(nbr.cpu().numpy(), ref)
    if name != "far":
        Xr = orc.features(pu.oracle_params(), w["env_offsets"], s, ref)
        assert np.max(np.abs(X.cpu().numpy() - Xr) / np.maximum(np.abs(Xr), 1.0)) < 1e-6

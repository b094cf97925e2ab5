"""Which HIP calls the library's host code makes, and on which device: run on a
CPU against a stand-in for the HIP runtime (fake_hip.cpp), in a process of its
own per scenario."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
fake = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
import numpy as np
from paper_2606_08039_amd import md

def log(clear=True):
    lines = fake.fake_log().decode().splitlines()
    if clear:
        fake.fake_log_clear()
    return lines

class T:
    # a tensor as far as the binding looks at one: an address nobody reads
    shape = (4096, 64)
    def data_ptr(self):
        return 4096

def state():
    return md.md_state(*[4096] * len(md.md_state._fields_))

def context(sizes, act=None, mask=7):
    c = md.md_create(md.md_default_params_cf2x(), 1 / 240, mask, md.MD_ACT_PID if act is None else act, 1)
    md.md_bind_layout(c, np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    return c

def kernels(lines):
    return [l.split()[2] for l in lines if "launch" in l]

LANES = ("ELi4ELi1ELi5", "ELi8ELi1ELi5")  # the step kernel's template arguments: lanes, unroll, sweep

def lanes(names):
    return [any(x in n for x in LANES) for n in names]

# a clock for the tuner: launches of several lanes take `fast`, others `slow`
CLOCK = ctypes.CFUNCTYPE(ctypes.c_float)
def clock(fast, slow):
    def ms():
        return fast if lanes([kernels(log(False))[-1]])[0] else slow
    f = CLOCK(ms)
    fake.fake_clock(f)
    return f

def tune(c, cache="", n_steps=10):
    ms = state()
    md.check(md.lib().md_autotune(c, ctypes.byref(ms), 4096, 0, n_steps, 0, 0, cache.encode(), 0), c)

def step(c, n=1, obs=None):
    md.md_step(c, state(), T(), False, obs, 1 if obs is not None else 0, n, 0, stream=0)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", so])

    def run(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE % so + code], cwd=ROOT, capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return run


def test_network_parameters_are_packed_on_the_network_s_device(fake):
    fake("""
fake.hipSetDevice(1)
m = md.md_mlp_create(64)
fake.hipSetDevice(0)
log()
md.md_mlp_set_params(m, np.zeros(md.MLP_NPARAMS, np.float32))
launches = [l for l in log() if "launch" in l]
assert launches and all(l.startswith("1 launch") for l in launches), launches
dev = ctypes.c_int(-1)
fake.hipGetDevice(ctypes.byref(dev))
assert dev.value == 0  # the caller's device again
""")


LAYOUTS = {"eight_lanes": "[32] * 20", "four_lanes": "[8, 5, 2] * 900", "one_lane": "[32] * 2000",
           "blocks": "[160, 31, 7]", "single": "[1] * 300"}
SETTERS = {
    "wind": "md.md_set_wind(c, models=md.MD_WIND_CONSTANT, v_mean=(0.1, 0.0, 0.0))",
    "wind_off": "md.md_set_wind(c, models=0)",
    "rk4": "md.md_set_integrator(c, md.MD_INTEG_RK4)",
    "euler": "md.md_set_integrator(c, md.MD_INTEG_EULER)",
    "dr": "d = md.md_dr(4096, None, None, 0.0, 0.0, 0.0, 0.0, 1, None, None)\n"
          "md.check(md.lib().md_set_domain_randomization(c, ctypes.byref(d)), c)",
    "dr_off": "md.md_set_domain_randomization(c, None)",
}


@pytest.mark.parametrize("name", list(LAYOUTS))
@pytest.mark.parametrize("first", ["", "wind", "rk4", "dr"])
def test_no_call_after_binding_allocates(fake, name, first):
    """Whatever is switched on or off after binding, a step (which a caller may
    be capturing) finds its tables: no allocation and no copy."""
    off = {"": "", "wind": "wind_off", "rk4": "euler", "dr": "dr_off"}
    code = "c = md.md_create(md.md_default_params_cf2x(), 1 / 240, 7, md.MD_ACT_PID, 1)\n"
    code += SETTERS.get(first, "") + "\n"
    code += "md.md_bind_layout(c, np.concatenate([[0], np.cumsum(%s)]).astype(np.int32))\nlog()\n" % LAYOUTS[name]
    for s in ("", off[first], "wind", "wind_off", "rk4", "euler", "dr", "dr_off"):
        code += SETTERS.get(s, "") + """
step(c)
md.md_datagen(c, state(), 7, T(), T(), stream=0)
calls = log()
assert sum("launch" in l for l in calls) == 2 and len(calls) == 2, (%r, calls)
""" % s
    fake(code)


def test_the_tuner_measures_the_default_plan_and_may_keep_it(fake, tmp_path):
    cache = str(tmp_path / "tune.json")
    fake("""
c = context([32] * 20)
cfg = md.md_get_launch_config(c)
keep = clock(1.0, 2.0)
tune(c, %r)
seen = lanes(kernels(log()))
assert any(seen) and not all(seen)
step(c)
assert lanes(kernels(log())) == [True]
assert md.md_get_launch_config(c) == cfg
# another context takes the cached choice
d = context([32] * 20)
md.md_set_launch_config(d, lanes_per_drone=1, unroll=1, waves_per_group=1)
log()
tune(d, %r)
assert not kernels(log())
step(d)
assert lanes(kernels(log())) == [True]
# and where another is faster, that one
keep = clock(2.0, 1.0)
tune(c)
log()
step(c)
assert lanes(kernels(log())) == [False]
""" % (cache, cache))


def test_a_choice_cached_before_the_default_had_lanes_is_measured_again(fake, tmp_path):
    cache = str(tmp_path / "tune.json")
    fake("""
import json
c = context([32] * 20)
keep = clock(1.0, 2.0)
tune(c, %r)
rec = json.load(open(%r))
old = dict(rec[0], lpd=4, unroll=1, waves=2, sym=0)
old["sig"] = old["sig"].replace("_lanes", "")
assert old["sig"] != rec[0]["sig"]
open(%r, "w").write("[\\n" + json.dumps(old) + "\\n]\\n")
d = context([32] * 20)
log()
tune(d, %r)
assert kernels(log())
step(d)
assert lanes(kernels(log())) == [True]
""" % ((cache,) * 4))


def test_the_default_configuration_set_or_kept_stays_the_default(fake):
    fake("""
for sizes in ([32] * 20, [8, 5, 2] * 900):
    c = context(sizes)
    md.md_set_launch_config(c, **md.md_get_launch_config(c))
    tune(c, n_steps=0)
    log()
    step(c)
    assert lanes(kernels(log())) == [True]
    # another unroll is the caller's own one-lane configuration
    md.md_set_launch_config(c, lanes_per_drone=1, unroll=2, waves_per_group=1)
    step(c)
    assert lanes(kernels(log())) == [False]
""")


def test_groups_of_the_rotation_sweep(fake):
    """One wave per workgroup unless the launch is long, stores rows and fills
    the 256 CUs evenly; never more threads than the configuration names, and
    every wave of the bins is launched."""
    fake("""
WIND, RK4, DR = "wind", "rk4", "dr"
def blocks(envs, m, steps, waves, what=None, rows=True):
    c = context([m] * envs)
    if what == WIND:
        md.md_set_wind(c, models=md.MD_WIND_CONSTANT, v_mean=(0.1, 0.0, 0.0))
    if what == RK4:
        md.md_set_integrator(c, md.MD_INTEG_RK4)
    if what == DR:
        d = md.md_dr(4096, None, None, 0.0, 0.0, 0.0, 0.0, 1, None, None)
        md.check(md.lib().md_set_domain_randomization(c, ctypes.byref(d)), c)
    md.md_set_launch_config(c, lanes_per_drone=1, unroll=1, waves_per_group=waves, pair_symmetric=3)
    log()
    step(c, steps, T() if rows else None)
    grid, block = [int(x) for x in [l for l in log() if "launch" in l][0].split()[3:5]]
    need = -(-envs * m // 64)
    assert need * 64 <= grid * block < (need + waves) * 64, (grid, block)
    md.md_destroy(c)
    return block // 64
for args, want in [((8192, 32, 500, 16), 16), ((8192, 32, 499, 16), 1), ((8192, 32, 500, 8), 1),
                   ((8192, 32, 500, 16, None, False), 1), ((6500, 32, 1000, 16), 16), ((6144, 32, 1000, 16), 1),
                   ((6146, 32, 1000, 16), 16), ((8193, 32, 1000, 16), 1), ((12000, 32, 1000, 16), 1),
                   ((16384, 32, 1000, 16), 16), ((4096, 64, 1000, 16), 16), ((16384, 16, 1000, 16), 16),
                   ((100, 32, 1000, 16), 1), ((8192, 32, 1000, 16, WIND), 16), ((8192, 32, 1000, 8, DR), 1),
                   ((8192, 32, 250, 16, RK4), 8), ((8192, 32, 249, 16, RK4), 1), ((8192, 32, 500, 8, RK4), 8), ((8192, 32, 500, 4, RK4), 1),
                   ((12000, 32, 500, 16, RK4), 8), ((10000, 32, 500, 16, RK4), 1), ((16384, 16, 500, 16, RK4), 1)]:
    got = blocks(*args)
    assert got == want, (args, got, want)
""")


def test_the_tuner_times_every_launch_once(fake):
    """Candidates that run the same kernel on the same workgroups are one, and a
    choice of the rotation sweep leaves longer launches their groups."""
    fake("""
def rotation_first():
    f = CLOCK(lambda: 1.0 if "ELi1ELi1ELi3" in kernels(log(False))[-1] else 2.0)
    fake.fake_clock(f)
    return f
for sizes in ([32] * 8192, [160, 31, 7], [2, 30, 17] * 3000, [64] * 50):
    c = context(sizes)
    log()
    keep = rotation_first()
    tune(c)
    first = [l for l in log() if "launch" in l]
    n = first.index(first[0], 1)  # the second round begins
    assert len(set(first[:n])) == n and first[:n] == first[n:2 * n], (sizes[0], first[:n])
    if sizes[0] in (32, 64):
        got = md.md_get_launch_config(c)
        assert got["pair_symmetric"] == 3 and got["waves_per_group"] == 16, got
""")

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

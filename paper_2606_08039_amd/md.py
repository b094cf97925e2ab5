"""ctypes binding of libmd (include/md.h), same names as the C ABI.

Argument marshalling only: every step of the simulation runs in the HIP
kernels of libmd.so.  PyTorch supplies device memory and streams.  If the
library is missing this module raises on first use -- there is no fallback.
"""
import ctypes
import os
import re
import struct

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libmd.so")
HEADER = os.path.join(os.path.dirname(HERE), "include", "md.h")

MD_OK = 0
MD_E_INVALID_ARG, MD_E_HIP, MD_E_OOM, MD_E_UNSUPPORTED, MD_E_LAYOUT = -1, -2, -3, -4, -5
MD_AERO_GND, MD_AERO_DRAG, MD_AERO_DW, MD_AERO_SURROGATE = 1, 2, 4, 8
MD_ACT_RPM, MD_ACT_PID, MD_ACT_VEL, MD_ACT_ATTITUDE, MD_ACT_DSL = 0, 1, 2, 3, 4
MD_INTEG_EULER, MD_INTEG_RK4 = 0, 1
ACTION_ROWS = {MD_ACT_RPM: 4, MD_ACT_PID: 4, MD_ACT_VEL: 4, MD_ACT_ATTITUDE: 4, MD_ACT_DSL: 7}
OBS_DIM = 20
STATE_ROWS = (("p", 3), ("q", 4), ("v", 3), ("w", 3), ("pid_int", 6), ("rpm", 4), ("ctl", 4))


class MdError(RuntimeError):
    def __init__(self, status, msg):
        super().__init__("libmd error %d: %s" % (status, msg))
        self.status = status


class md_params(ctypes.Structure):
    _fields_ = [(n, ctypes.c_double) for n in (
        "m", "L", "kf", "km", "Ixx", "Iyy", "Izz", "thrust2weight", "r_p", "g",
        "C_gnd", "c_xy", "c_z", "C1", "C2", "C3", "dw_dz_min")] + [
        ("pos_kp", ctypes.c_double * 3), ("pos_ki", ctypes.c_double * 3),
        ("pos_kd", ctypes.c_double * 3), ("pos_i_clamp", ctypes.c_double),
        ("att_kp", ctypes.c_double * 3), ("att_ki", ctypes.c_double * 3),
        ("att_kd", ctypes.c_double * 3), ("att_i_clamp", ctypes.c_double),
        ("dsl_pos_kp", ctypes.c_double * 3), ("dsl_pos_ki", ctypes.c_double * 3),
        ("dsl_pos_kd", ctypes.c_double * 3), ("dsl_pos_i_clamp", ctypes.c_double),
        ("dsl_att_kp", ctypes.c_double * 3), ("dsl_att_ki", ctypes.c_double * 3),
        ("dsl_att_kd", ctypes.c_double * 3), ("dsl_att_i_clamp", ctypes.c_double),
        ("dsl_max_speed", ctypes.c_double), ("dsl_max_yaw_rate", ctypes.c_double)]


class md_derived(ctypes.Structure):
    _fields_ = [(n, ctypes.c_double) for n in ("hover_rpm", "max_rpm", "max_thrust", "h_clip")]


class md_state(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("p", "q", "v", "w", "pid_int", "rpm", "ctl",
                                               "rpm_cmd", "act_hist", "act_count", "wind",
                                               "obs_hist", "obs_count")]


class md_wind(ctypes.Structure):
    _fields_ = [("models", ctypes.c_uint32), ("v_mean", ctypes.c_float * 3), ("rho", ctypes.c_float),
                ("cd_area", ctypes.c_float), ("gust_prob", ctypes.c_float), ("gust_duration", ctypes.c_float),
                ("gust_amp", ctypes.c_float), ("dryden_sigma", ctypes.c_float),
                ("dryden_airspeed", ctypes.c_float), ("sin_amp", ctypes.c_float), ("sin_omega", ctypes.c_float),
                ("seed", ctypes.c_uint64), ("v_mean_drone", ctypes.c_void_p)]


MD_WIND_CONSTANT, MD_WIND_GUST, MD_WIND_DRYDEN, MD_WIND_SINUSOIDAL = 1, 2, 4, 8
MD_WIND_COMBINED = 15


class md_dr(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("scale", "tau_mot", "delay")] + [
        (n, ctypes.c_float) for n in ("noise_p", "noise_v", "noise_rpy", "noise_w")] + [
        ("seed", ctypes.c_uint64), ("obs_delay", ctypes.c_void_p), ("obs_bias", ctypes.c_void_p)]


MD_DR_ROWS = ("m", "J", "L", "kf", "km", "drag", "C_gnd", "C1", "max_rpm", "g",
              "bias0", "bias1", "bias2", "bias3")
MD_DR_NSCALE, MD_DR_HIST, MD_DR_OBS_HIST = 14, 32, 8


_lib = None
_packed_step = None
_VP = ctypes.c_void_p


def lib():
    """The loaded libmd.so; raises if it has not been built."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError("libmd.so is not built (%s); run `python -m paper_2606_08039_amd.build`"
                           % LIB_PATH)
    # torch first: its HIP runtime and libmd's share one soname, so loading
    # libmd first would hand torch a runtime it was not built against (torch
    # then finds no GPU); loaded after torch, libmd binds to torch's runtime
    # and both use one set of devices, streams and allocations.
    import torch  # noqa: F401
    L = ctypes.CDLL(LIB_PATH)
    sig = {
        "md_version": (ctypes.c_char_p, []),
        "md_default_params_cf2x": (ctypes.c_int32, [ctypes.POINTER(md_params)]),
        "md_derive": (ctypes.c_int32, [ctypes.POINTER(md_params), ctypes.POINTER(md_derived)]),
        "md_create": (ctypes.c_int32, [ctypes.POINTER(md_params), ctypes.c_float, ctypes.c_uint32,
                                       ctypes.c_int, ctypes.c_int, ctypes.POINTER(_VP)]),
        "md_destroy": (None, [_VP]),
        "md_last_error": (ctypes.c_char_p, [_VP]),
        "md_bind_layout": (ctypes.c_int32, [_VP, ctypes.POINTER(ctypes.c_int32), ctypes.c_int,
                                            ctypes.c_int]),
        "md_step": (ctypes.c_int32, [_VP, ctypes.POINTER(md_state), _VP, ctypes.c_int, _VP,
                                     ctypes.c_int, ctypes.c_int, ctypes.c_int64, _VP]),
    }
    for name, (res, args) in sig.items():
        f = getattr(L, name)
        f.restype = res
        f.argtypes = args
    # the same function for a DeviceState's packed pointers (a second object:
    # callers of lib().md_step keep the check of its argument's type)
    global _packed_step
    _packed_step = L["md_step"]
    _packed_step.restype, _packed_step.argtypes = ctypes.c_int32, [_VP, ctypes.c_char_p] + sig["md_step"][1][2:]
    _lib = L
    _bind_extra(L)
    return L


def _bind_extra(L):
    """Signatures of the optional subsystems (autotuner, graphs, surrogate)."""
    from . import md_extra_sigs
    for name, (res, args) in md_extra_sigs.signatures().items():
        if hasattr(L, name):
            f = getattr(L, name)
            f.restype = res
            f.argtypes = args


def header_symbols():
    """Names of the functions include/md.h declares."""
    txt = re.sub(r"/\*.*?\*/", " ", open(HEADER).read(), flags=re.S)
    return sorted(set(re.findall(r"\b(md_[a-z0-9_]+)\s*\(", txt)))


def check(status, ctx=None):
    if status != MD_OK:
        msg = lib().md_last_error(ctx).decode()
        raise MdError(status, msg)


_current_raw_stream = None  # torch's current stream of the current device, as an address


def _stream_ptr(stream):
    # every call that steps, predicts or trains passes here: torch's own
    # Stream object costs more than the launch it would be used for
    if stream is None:
        global _current_raw_stream
        if _current_raw_stream is None:
            import torch
            torch.cuda.init()
            raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
            dev = getattr(torch._C, "_cuda_getDevice", None)
            if raw is None or dev is None:  # internals of torch, which another version may not have
                _current_raw_stream = lambda: torch.cuda.current_stream().cuda_stream  # noqa: E731
            else:
                _current_raw_stream = lambda: raw(dev())  # noqa: E731
        return _current_raw_stream()
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


_STATE_PTRS = struct.Struct("%dQ" % len(md_state._fields_))


# ------------------------------------------------------------------ C ABI

def md_version():
    return lib().md_version().decode()


def md_default_params_cf2x():
    p = md_params()
    check(lib().md_default_params_cf2x(ctypes.byref(p)))
    return p


def md_derive(params):
    d = md_derived()
    check(lib().md_derive(ctypes.byref(params), ctypes.byref(d)))
    return d


def md_create(params, dt, aero_mask, act_type, ctrl_decim=1):
    ctx = _VP()
    st = lib().md_create(ctypes.byref(params), float(dt), int(aero_mask), int(act_type),
                         int(ctrl_decim), ctypes.byref(ctx))
    check(st, None)
    return ctx


def md_destroy(ctx):
    lib().md_destroy(ctx)


def md_last_error(ctx):
    return lib().md_last_error(ctx).decode()


def md_bind_layout(ctx, env_offsets):
    off = np.ascontiguousarray(np.asarray(env_offsets, dtype=np.int32))
    st = lib().md_bind_layout(ctx, off.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)),
                              len(off) - 1, int(off[-1]))
    check(st, ctx)


def md_step(ctx, state, action, action_per_step, obs=None, n_obs_slots=0, n_steps=1, step0=0,
            stream=None):
    """state: DeviceState (or md_state); action/obs: CUDA float32 tensors."""
    step = lib().md_step
    if type(state) is DeviceState:
        step, s = _packed_step, state.pointers()
    else:
        s = ctypes.byref(state.as_md_state() if hasattr(state, "as_md_state") else state)
    st = step(ctx, s, action.data_ptr(), 1 if action_per_step else 0,
              None if obs is None else obs.data_ptr(), int(n_obs_slots),
              int(n_steps), int(step0), _stream_ptr(stream))
    if st != MD_OK:
        check(st, ctx)


# ------------------------------------------------------------------ device buffers

_STATE_KEYS = tuple(n for n, _ in md_state._fields_)


class DeviceState:
    """Float32 SoA state on the GPU, one torch tensor [rows][N] per field."""

    def __init__(self, n, device="cuda"):
        import torch
        self.n = n
        self.t = {k: torch.zeros((r, n), dtype=torch.float32, device=device) for k, r in STATE_ROWS}
        self.t["q"][0] = 1.0

    @classmethod
    def from_numpy(cls, s, device="cuda"):
        import torch
        n = s["p"].shape[1]
        d = cls(n, device)
        for k, _ in STATE_ROWS:
            if k in s:
                d.t[k].copy_(torch.from_numpy(np.ascontiguousarray(s[k], dtype=np.float32)))
        return d

    def add_dr_blocks(self, act_type, s=None):
        """The blocks the domain-randomised step needs: the held controller
        command (from s["rpm_cmd"], else the rotor speeds), the action and
        sensor latency rings and their fill counts (from s, else empty)."""
        import torch
        rows = ACTION_ROWS[act_type]
        dev = self.t["p"].device
        self.t["rpm_cmd"] = self.t["rpm"].clone()
        self.t["act_hist"] = torch.zeros((MD_DR_HIST, rows, self.n), dtype=torch.float32, device=dev)
        self.t["act_count"] = torch.zeros(self.n, dtype=torch.int32, device=dev)
        self.t["obs_hist"] = torch.zeros((MD_DR_OBS_HIST, 20, self.n), dtype=torch.float32, device=dev)
        self.t["obs_count"] = torch.zeros(self.n, dtype=torch.int32, device=dev)
        if s is not None:
            for k, dt in (("rpm_cmd", np.float32), ("act_hist", np.float32), ("act_count", np.int32),
                          ("obs_hist", np.float32), ("obs_count", np.int32)):
                if k in s:
                    self.t[k].copy_(torch.from_numpy(np.ascontiguousarray(s[k], dtype=dt)))
        return self

    def add_wind_block(self, s=None):
        """The wind state block (Dryden velocity 0, gusts idle, or s["wind"])."""
        import torch
        w = torch.zeros((5, self.n), dtype=torch.float32, device=self.t["p"].device)
        w[3] = -1.0
        if s is not None and "wind" in s:
            w.copy_(torch.from_numpy(np.ascontiguousarray(s["wind"], dtype=np.float32)))
        self.t["wind"] = w
        return self

    def to_numpy(self):
        return {k: v.cpu().numpy() for k, v in self.t.items()}

    def clone(self):
        d = DeviceState.__new__(DeviceState)
        d.n = self.n
        d.t = {k: v.clone() for k, v in self.t.items()}
        return d

    def as_md_state(self):
        return md_state.from_buffer_copy(self.pointers())

    def pointers(self):
        """The bytes of as_md_state(): the blocks' addresses as they are now."""
        t = self.t
        return _STATE_PTRS.pack(*[t[k].data_ptr() if k in t else 0 for k in _STATE_KEYS])


# ------------------------------------------------------------------ surrogate network

MLP_IN, MLP_HIDDEN, MLP_OUT, MLP_NPARAMS, MLP_NORM = 64, 128, 6, 42118, 140
MLP_SHAPES = ((128, 64), (128,), (128, 128), (128,), (128, 128), (128,), (6, 128), (6,))


def _fptr(a):
    assert a.dtype == np.float32 and a.flags.c_contiguous
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_float))


def mlp_check(status, m):
    if status != MD_OK:
        raise MdError(status, lib().md_mlp_last_error(m).decode())


def md_mlp_create(max_batch):
    m = _VP()
    st = lib().md_mlp_create(int(max_batch), ctypes.byref(m))
    if st != MD_OK:
        raise MdError(st, "md_mlp_create")
    return m


def md_mlp_destroy(m):
    lib().md_mlp_destroy(m)


def md_mlp_set_params(m, flat):
    a = np.ascontiguousarray(flat, dtype=np.float32)
    assert a.size == MLP_NPARAMS
    mlp_check(lib().md_mlp_set_params(m, _fptr(a)), m)


def md_mlp_get_params(m):
    a = np.zeros(MLP_NPARAMS, dtype=np.float32)
    mlp_check(lib().md_mlp_get_params(m, _fptr(a)), m)
    return a


def md_mlp_set_norm(m, norm):
    a = np.ascontiguousarray(norm, dtype=np.float32)
    assert a.size == MLP_NORM
    mlp_check(lib().md_mlp_set_norm(m, _fptr(a)), m)


def md_mlp_get_norm(m):
    a = np.zeros(MLP_NORM, dtype=np.float32)
    mlp_check(lib().md_mlp_get_norm(m, _fptr(a)), m)
    return a


def md_mlp_forward(m, X, B=None, Y=None, stream=None):
    B = X.shape[0] if B is None else int(B)
    st = lib().md_mlp_forward(m, X.data_ptr(), B, None if Y is None else Y.data_ptr(), _stream_ptr(stream))
    if st != MD_OK:
        mlp_check(st, m)


MD_MLP_NOALLOC_MAX_BATCH = 4096


def md_mlp_forward_noalloc(m, X, Y, B=None, stream=None):
    """md_mlp_forward with its intermediates on chip (allocates nothing, keeps
    nothing); Y [B][6] float32 receives the outputs."""
    B = X.shape[0] if B is None else int(B)
    st = lib().md_mlp_forward_noalloc(m, X.data_ptr(), B, Y.data_ptr(), _stream_ptr(stream))
    if st != MD_OK:
        mlp_check(st, m)


def md_mlp_backward(m, T, B=None, stream=None):
    B = T.shape[0] if B is None else int(B)
    st = lib().md_mlp_backward(m, T.data_ptr(), B, _stream_ptr(stream))
    if st != MD_OK:
        mlp_check(st, m)


def md_mlp_get_grads(m):
    a = np.zeros(MLP_NPARAMS, dtype=np.float32)
    mlp_check(lib().md_mlp_get_grads(m, _fptr(a)), m)
    return a


def md_mlp_loss(m):
    d = ctypes.c_double()
    mlp_check(lib().md_mlp_loss(m, ctypes.byref(d)), m)
    return d.value


def md_mlp_adam(m, lr, beta1=0.9, beta2=0.999, eps=1e-8, stream=None):
    mlp_check(lib().md_mlp_adam(m, float(lr), float(beta1), float(beta2), float(eps),
                                _stream_ptr(stream)), m)


def mlp_unflatten(flat):
    """Split the flat parameter vector into W1, b1, ..., W4, b4."""
    out, o = [], 0
    for sh in MLP_SHAPES:
        n = int(np.prod(sh))
        out.append(np.asarray(flat[o:o + n]).reshape(sh))
        o += n
    return out


def mlp_flatten(parts):
    return np.concatenate([np.asarray(p, dtype=np.float32).ravel() for p in parts])


# ------------------------------------------------------------------ surrogate in the step

class md_judge(ctypes.Structure):
    _fields_ = [(n, ctypes.c_double) for n in ("n_judged", "force_err2", "force_ref2", "torque_err2",
                                                "n_fallback", "n_drone_steps", "force_rel_err",
                                                "n_nonfinite", "n_knn_full")]


def md_load_surrogate(ctx, flat, norm, dz_ood=1e-3, judge_stride=64):
    a = np.ascontiguousarray(flat, dtype=np.float32)
    b = np.ascontiguousarray(norm, dtype=np.float32)
    assert a.size == MLP_NPARAMS and b.size == MLP_NORM
    check(lib().md_load_surrogate(ctx, _fptr(a), _fptr(b), float(dz_ood), int(judge_stride)), ctx)


def md_load_surrogate_mlp(ctx, m, dz_ood=1e-3, judge_stride=64):
    check(lib().md_load_surrogate_mlp(ctx, m, float(dz_ood), int(judge_stride)), ctx)


def md_datagen(ctx, state, aero_mask, X, Y, nbr=None, stream=None):
    ms = state.as_md_state() if hasattr(state, "as_md_state") else state
    check(lib().md_datagen(ctx, ctypes.byref(ms), int(aero_mask), _VP(X.data_ptr()), _VP(Y.data_ptr()),
                           _VP(nbr.data_ptr()) if nbr is not None else None, _stream_ptr(stream)), ctx)


def md_judge_stats(ctx):
    j = md_judge()
    check(lib().md_judge_stats(ctx, ctypes.byref(j)), ctx)
    return {k: getattr(j, k) for k, _ in md_judge._fields_}


def md_set_surrogate_ood(ctx, max_speed=0.0, max_rel_speed=0.0, max_tilt=0.0):
    check(lib().md_set_surrogate_ood(ctx, float(max_speed), float(max_rel_speed), float(max_tilt)), ctx)


def md_set_surrogate_region(ctx, near_dz=0.0, near_r=0.0, far_dz=0.0):
    check(lib().md_set_surrogate_region(ctx, float(near_dz), float(near_r), float(far_dz)), ctx)


def md_set_surrogate_knn_reuse(ctx, reuse=True):
    check(lib().md_set_surrogate_knn_reuse(ctx, int(bool(reuse))), ctx)


def md_judge_reset(ctx):
    check(lib().md_judge_reset(ctx), ctx)


# ------------------------------------------------------------------ domain randomisation

def md_set_domain_randomization(ctx, scale=None, tau_mot=None, delay=None, noise=(0.0, 0.0, 0.0, 0.0),
                                seed=0, obs_delay=None, obs_bias=None):
    """scale: CUDA float32 [MD_DR_NSCALE][N]; tau_mot: float32 [N] or None;
    delay: int32 [N] or None; noise: sensor noise sigmas (position,
    velocity, roll/pitch/yaw, body rates); seed: Philox key of the noise;
    obs_delay: int32 [N] sensor latency in steps, or None; obs_bias: float32
    [12][N] sticky bias on the p, v, rpy, w rows, or None.  scale None turns
    randomisation off.  The tensors must stay alive while the context uses
    them."""
    if scale is None:
        check(lib().md_set_domain_randomization(ctx, None), ctx)
        return
    import torch
    assert scale.dtype == torch.float32 and scale.is_contiguous()
    assert tau_mot is None or (tau_mot.dtype == torch.float32 and tau_mot.is_contiguous())
    assert delay is None or (delay.dtype == torch.int32 and delay.is_contiguous())
    assert obs_delay is None or (obs_delay.dtype == torch.int32 and obs_delay.is_contiguous())
    assert obs_bias is None or (obs_bias.dtype == torch.float32 and obs_bias.is_contiguous())
    nz = [float(x) for x in noise]
    d = md_dr(scale.data_ptr(), tau_mot.data_ptr() if tau_mot is not None else None,
              delay.data_ptr() if delay is not None else None, nz[0], nz[1], nz[2], nz[3], int(seed),
              obs_delay.data_ptr() if obs_delay is not None else None,
              obs_bias.data_ptr() if obs_bias is not None else None)
    check(lib().md_set_domain_randomization(ctx, ctypes.byref(d)), ctx)


# ------------------------------------------------------------------ wind

def md_set_wind(ctx, models=0, v_mean=(0.0, 0.0, 0.0), rho=1.225, cd_area=0.01, gust_prob=0.0,
                gust_duration=0.5, gust_amp=0.0, dryden_sigma=0.0, dryden_airspeed=1.0, sin_amp=0.0,
                sin_omega=0.0, seed=0, v_mean_drone=None):
    """models 0 turns wind off.  v_mean_drone: CUDA float32 [3][N] per-drone
    mean wind replacing v_mean, or None; it must stay alive while the
    context uses it."""
    if not models:
        check(lib().md_set_wind(ctx, None), ctx)
        return
    if v_mean_drone is not None:
        import torch
        assert v_mean_drone.dtype == torch.float32 and v_mean_drone.is_contiguous()
    w = md_wind(int(models), (ctypes.c_float * 3)(*v_mean), rho, cd_area, gust_prob, gust_duration, gust_amp,
                dryden_sigma, dryden_airspeed, sin_amp, sin_omega, int(seed),
                v_mean_drone.data_ptr() if v_mean_drone is not None else None)
    check(lib().md_set_wind(ctx, ctypes.byref(w)), ctx)


# ------------------------------------------------------------------ integrator

def md_set_integrator(ctx, integrator):
    check(lib().md_set_integrator(ctx, int(integrator)), ctx)


def md_get_integrator(ctx):
    v = ctypes.c_int(-1)
    check(lib().md_get_integrator(ctx, ctypes.byref(v)), ctx)
    return v.value


# ------------------------------------------------------------------ launch configuration, graphs

class md_launch_config(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("lanes_per_drone", "unroll", "waves_per_group",
                                            "pair_symmetric")]


def md_get_launch_config(ctx):
    c = md_launch_config()
    check(lib().md_get_launch_config(ctx, ctypes.byref(c)), ctx)
    return {k: getattr(c, k) for k, _ in md_launch_config._fields_}


def md_set_launch_config(ctx, lanes_per_drone=1, unroll=4, waves_per_group=1, pair_symmetric=0):
    c = md_launch_config(lanes_per_drone, unroll, waves_per_group, pair_symmetric)
    check(lib().md_set_launch_config(ctx, ctypes.byref(c)), ctx)


def md_autotune(ctx, state, action, action_per_step, n_steps=20, step0=0, stream=None,
                cache_path=None, force=False):
    ms = state.as_md_state() if hasattr(state, "as_md_state") else state
    cp = cache_path.encode() if cache_path is not None else None
    check(lib().md_autotune(ctx, ctypes.byref(ms), _VP(action.data_ptr()), int(bool(action_per_step)),
                            int(n_steps), int(step0), _stream_ptr(stream), cp, int(bool(force))), ctx)
    return md_get_launch_config(ctx)


def md_autotune_obs(ctx, state, action, action_per_step, obs, n_obs_slots, n_steps=20, step0=0, stream=None,
                    cache_path=None, force=False):
    ms = state.as_md_state() if hasattr(state, "as_md_state") else state
    cp = cache_path.encode() if cache_path is not None else None
    check(lib().md_autotune_obs(ctx, ctypes.byref(ms), _VP(action.data_ptr()), int(bool(action_per_step)),
                                _VP(obs.data_ptr()) if obs is not None else None, int(n_obs_slots),
                                int(n_steps), int(step0), _stream_ptr(stream), cp, int(bool(force))), ctx)
    return md_get_launch_config(ctx)


def md_rollout_graph_create(ctx, state, action, action_per_step, obs=None, n_obs_slots=0,
                            steps_per_launch=1, n_launches=1, step0=0, stream=None):
    ms = state.as_md_state() if hasattr(state, "as_md_state") else state
    g = _VP()
    check(lib().md_rollout_graph_create(ctx, ctypes.byref(ms), _VP(action.data_ptr()),
                                        int(bool(action_per_step)),
                                        _VP(obs.data_ptr()) if obs is not None else None,
                                        int(n_obs_slots), int(steps_per_launch), int(n_launches),
                                        int(step0), _stream_ptr(stream), ctypes.byref(g)), ctx)
    g._md_state = ms  # the captured kernels hold these device pointers
    return g


def md_graph_launch(g, stream=None):
    st = lib().md_graph_launch(g, _stream_ptr(stream))
    if st != MD_OK:
        raise MdError(st, "md_graph_launch")


def md_graph_destroy(g):
    lib().md_graph_destroy(g)

"""The binding's md_step: what it takes for a state and what it refuses, and the
stream it finds, on the CPU (no call reaches a GPU: a context that is null
returns MD_E_INVALID_ARG)."""
import ctypes

import pytest

from paper_2606_08039_amd import md


class Address:
    def data_ptr(self):
        return 4096


def test_lib_md_step_takes_a_state_only():
    L = md.lib()
    rest = (4096, 0, None, 0, 1, 0, None)
    s = md.md_state()
    for state in (s, ctypes.byref(s), ctypes.pointer(s)):
        assert L.md_step(None, state, *rest) == md.MD_E_INVALID_ARG
    for other in (md.md_params(), ctypes.byref(md.md_params()), 4096, b"state"):
        with pytest.raises(ctypes.ArgumentError):
            L.md_step(None, other, *rest)


def test_md_step_takes_states_and_objects_that_make_one():
    def step(state):
        with pytest.raises(md.MdError) as ei:
            md.md_step(None, state, Address(), False, stream=0)
        assert ei.value.status == md.MD_E_INVALID_ARG

    class Own(md.DeviceState):
        made = 0

        def __init__(self):
            self.t = {}

        def as_md_state(self):
            Own.made += 1
            return md.md_state()

    step(md.md_state())
    step(Own())
    assert Own.made == 1  # a subclass's own as_md_state is the one that counts
    plain = md.DeviceState.__new__(md.DeviceState)
    plain.t = {"p": Address()}
    step(plain)
    assert plain.as_md_state().p == 4096 and not plain.as_md_state().q
    with pytest.raises(ctypes.ArgumentError):
        md.md_step(None, md.md_params(), Address(), False, stream=0)


def test_stream_without_torch_s_internals(monkeypatch):
    import torch

    class Internals:
        pass

    class Stream:
        cuda_stream = 77
    monkeypatch.setattr(md, "_current_raw_stream", None)
    monkeypatch.setattr(torch, "_C", Internals())
    monkeypatch.setattr(torch.cuda, "init", lambda: None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream())
    assert md._stream_ptr(None) == 77
    assert md._stream_ptr(5) == 5 and md._stream_ptr(Stream()) == 77

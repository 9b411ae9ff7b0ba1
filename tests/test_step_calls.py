"""The extension module behind Python's step calls fills the argument structs as the ctypes structures do, and takes nothing else.
Callbacks stand for the library's entry points."""
import ctypes as C
import dataclasses
import importlib.machinery
import os
import sys

import numpy as np
import pytest
import torch

from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd import build

from paper_2105_05720_amd import _step_calls as native
T = [torch.zeros(8, dtype=torch.float16) for _ in range(20)]
HP = cc.Hyper(lr=0.1, beta1=0.5, beta2=1 / 3, eps=1e-30, loss_scale=7, step=2**31 - 1, grad_average=-1, adam_mode=True, skip_mode=3)


@pytest.fixture(autouse=True)
def bound():
    assert native.bind(cc.Plan, cc.Hyper, cc.Tensor, torch.Tensor, torch.nn.Parameter, lambda: 3, lambda device: 1000 + device)
    yield
    if cc._torch is not None:
        cc._bind_native()


class Seen:
    """A function of the library's signature that keeps what it was called with."""

    def __init__(self, *sizes, rc=0):        # a struct's size, or 0 for a plain word
        self.args, self.sizes, self.rc = None, sizes, rc
        self.fn = C.CFUNCTYPE(C.c_int, *[C.c_void_p] * len(sizes))(self)
        self.at = C.cast(self.fn, C.c_void_p).value

    def __call__(self, *args):
        self.args = [C.string_at(a, n) if n else a for a, n in zip(args, self.sizes)]
        return self.rc


def plan(handle):
    p = cc.Plan(0, [])
    p.handle = handle
    return p


@pytest.mark.parametrize("flag,where", [(T[0], T[0].data_ptr()), (2**63, 2**63), (torch.nn.Parameter(T[1]), T[1].data_ptr())], ids=["tensor", "address", "parameter"])
@pytest.mark.parametrize("hp", [cc.Hyper(), HP, cc.Hyper(lr=float("inf"), beta1=float("nan"), step=-2**31)], ids=["defaults", "odd", "not finite"])
def test_step(hp, flag, where):
    seen = Seen(0, C.sizeof(cc.cc_hparams), 0, 0, rc=-4)
    p = plan(1 << 40)
    assert native.step(seen.at, p, hp, flag, None) == -4
    p.handle = None
    assert seen.args == [1 << 40, bytes(hp.to_c()), where, 1003]


@pytest.mark.parametrize("slices", [(), T[:1], tuple(T[:16]), T])
def test_static_step(slices):
    t = cc.Tensor(5, T[0], T[1], T[2], T[3], T[4], T[5], T[6], slices, 0.25)
    seen = Seen(C.sizeof(cc.cc_tensor), 0, C.sizeof(cc.cc_hparams), 0, 0)
    assert native.static_step(seen.at, t, len(slices), HP, T[7], None) == 0
    got, want = seen.args[0], bytes(cc._c_tensor(t))
    assert got == want and (seen.args[1] or 0) & 0xffffffff == len(slices) and seen.args[2:] == [bytes(HP.to_c()), T[7].data_ptr(), 1003]


@pytest.mark.parametrize("numel,slices", [(None, T[:1]), (3, T[:16]), (0, tuple(T))])
def test_epilogue(numel, slices):
    seen = Seen(C.sizeof(cc.cc_epilogue), 0)
    args = (slices, T[1], T[2], T[3], 2**40, 4096, 0.3, 2**64 - 1)
    assert native.epilogue(seen.at, *args, None, numel) == 0
    assert seen.args == [bytes(cc._epilogue(*args, numel)), 1003]


class Sub(torch.Tensor):
    pass


class Own(cc.Hyper):
    pass


@pytest.mark.parametrize("hp", [dataclasses.replace(cc.Hyper(), **{k: v}) for k, v in (
    ("step", 2**31), ("step", -2**31 - 1), ("step", 1.0), ("adam_mode", np.int32(1)), ("lr", 1e39), ("lr", 10**400), ("eps", "x"), ("beta1", None), ("lr", np.float32(1)))]
    + [Own(), cc.Hyper().to_c(), None])
def test_hyper_parameters_that_are_left_to_the_ctypes_structure(hp):
    seen = Seen(0, 0, 0, 0)
    assert native.step(seen.at, plan(0), hp, T[0], None) == 1 and seen.args is None


def test_other_arguments_that_are_left_to_the_general_path():
    seen, hp = Seen(0, 0, 0, 0, 0), cc.Hyper()
    missing = cc.Hyper()
    del missing.__dict__["lr"]                                   # the class's default holds then
    sub = torch.Tensor._make_subclass(Sub, T[0])
    for p, h, flag, stream in ((plan(None), hp, T[0], None), (object(), hp, T[0], None), (plan(0), missing, T[0], None), (plan(0), hp, sub, None),
                               (plan(0), hp, None, None), (plan(0), hp, -1, None), (plan(0), hp, T[0], 0)):
        assert native.step(seen.at, p, h, flag, stream) == 1
    good = dict(numel=5, w_in=T[0], m_in=T[1], v_in=T[2], w_out=T[3], m_out=T[4], v_out=T[5], w16_out=T[6], grad=T[:2])
    for k, v in (("numel", -1), ("numel", 2**64), ("w_in", 16), ("v_out", None), ("w16_out", sub), ("grad", [T[0], 16]), ("grad", iter(T)), ("grad", None), ("weight_decay", "x")):
        assert native.static_step(seen.at, cc.Tensor(**dict(good, **{k: v})), 2, hp, T[0], None) == 1
    assert native.static_step(seen.at, cc.Tensor(**good), 2.0, hp, T[0], None) == 1
    call = [T[:2], T[0], T[1], T[2], 0, 8, 0.1, 1, None, None]
    for i, v in ((0, [T[0], sub]), (1, 16), (2, None), (3, sub), (4, -8), (5, 2**32), (6, "x"), (7, -1), (8, 5), (9, 2.5)):
        assert native.epilogue(seen.at, *(v if i == j else x for j, x in enumerate(call))) == 1
    assert seen.args is None


def test_a_torch_function_mode_sees_the_tensors():
    from torch.overrides import TorchFunctionMode

    class Mode(TorchFunctionMode):
        asked = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            Mode.asked += func is torch.Tensor.data_ptr
            return func(*args, **(kwargs or {}))
    seen = Seen(0, 0, 0, 0)
    with Mode():
        assert native.step(seen.at, plan(0), cc.Hyper(), T[0], None) == 0
    assert Mode.asked == 1


@pytest.fixture
def first_call(monkeypatch):
    """As before the process's first step call, on a machine with a device."""
    for name in ("_torch", "_raw_stream"):
        monkeypatch.setattr(cc, name, None)
    for name in ("_native_step", "_native_static", "_native_epilogue"):
        monkeypatch.setattr(cc, name, cc._not_taken)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 70 + device, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 2, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 2)


def test_without_the_module_the_calls_say_so_once_and_go_through_ctypes(first_call, monkeypatch, recwarn):
    import paper_2105_05720_amd as package
    monkeypatch.setitem(sys.modules, package.__name__ + "._step_calls", None)
    monkeypatch.delattr(package, "_step_calls", raising=False)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert cc._current_stream() == 72
    recwarn.clear()
    assert cc._current_stream() == 72 and not recwarn.list
    assert cc._native_step is cc._native_static is cc._native_epilogue is cc._not_taken


def test_a_first_call_that_finds_no_device_is_not_the_last_to_look(first_call, monkeypatch):
    with monkeypatch.context() as m:
        m.setattr(torch.cuda, "current_device", lambda: (_ for _ in ()).throw(RuntimeError("no device")))
        for _ in range(2):
            with pytest.raises(RuntimeError, match="no device"):
                cc._current_stream()
    assert cc._current_stream() == 72 and cc._native_step is native.step


def test_the_module_is_built_for_one_python_and_the_library_without_it(monkeypatch, tmp_path, capsys):
    assert build.STEP_CALLS.endswith(importlib.machinery.EXTENSION_SUFFIXES[0]) and native.__file__ == build.STEP_CALLS
    monkeypatch.setattr(build, "STEP_CALLS", str(tmp_path / "module.so"))
    monkeypatch.setattr(build, "is_stale", lambda: False)
    monkeypatch.setenv("PATH", str(tmp_path))                    # no compiler
    assert build.build_library(force=False) == build.LIB
    assert "not built" in capsys.readouterr().err and not os.path.exists(build.STEP_CALLS)

"""Thin ctypes layer over libccfused.so: same names as include/ccfused.h, argument marshalling only.

Device buffers are torch tensors (or raw integer device addresses); every step of the update runs in the
library's kernels.  The library is loaded on first use and a missing build raises: there is no fallback.
"""
from __future__ import annotations

import ctypes as C
import os
import struct
import warnings
from dataclasses import dataclass, field
from typing import List, Optional, Sequence

CC_MAX_R = 16
CC_GRAD_F16, CC_GRAD_F32 = 0, 1
CC_SCHEDULE_AUTO, CC_SCHEDULE_PER_CHUNK, CC_SCHEDULE_ORDERED = 0, 1, 2
CC_CACHE_AUTO, CC_CACHE_STREAMING, CC_CACHE_RESIDENT, CC_CACHE_WRITE_THROUGH = 0, 1, 2, 3
CC_OK, CC_ERR_NULL, CC_ERR_ARG, CC_ERR_ALIGN, CC_ERR_ALIAS, CC_ERR_HIP, CC_ERR_NOMEM = 0, -1, -2, -3, -4, -5, -6

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libccfused.so")
_lib = None
_at = {}           # the addresses of the calls that a training step makes
_packed = {}       # the calls that a training step makes, typed to take their argument structs as packed bytes (see _step)


class CcError(RuntimeError):
    def __init__(self, code: int, message: str):
        super().__init__("ccfused error %d: %s" % (code, message))
        self.code = code


class cc_tensor(C.Structure):
    _fields_ = [("numel", C.c_uint64),
                ("w_in", C.c_void_p), ("m_in", C.c_void_p), ("v_in", C.c_void_p),
                ("w_out", C.c_void_p), ("m_out", C.c_void_p), ("v_out", C.c_void_p),
                ("w16_out", C.c_void_p),
                ("grad", C.c_void_p * CC_MAX_R),
                ("weight_decay", C.c_float)]


class cc_hparams(C.Structure):
    _fields_ = [("lr", C.c_float), ("beta1", C.c_float), ("beta2", C.c_float), ("eps", C.c_float),
                ("loss_scale", C.c_float), ("step", C.c_int32), ("grad_average", C.c_int32),
                ("adam_mode", C.c_int32), ("skip_mode", C.c_int32)]


class cc_epilogue(C.Structure):
    _fields_ = [("numel", C.c_uint64), ("first", C.c_uint64), ("hidden", C.c_uint32), ("R", C.c_int32),
                ("partial", C.c_void_p * CC_MAX_R), ("bias", C.c_void_p), ("residual", C.c_void_p), ("out", C.c_void_p),
                ("dropout_p", C.c_float), ("seed", C.c_uint64)]


# every symbol include/ccfused.h declares
EXPORTS = {
    "cc_chunk_count": (C.c_int64, [C.POINTER(C.c_uint64), C.c_int32, C.c_int32]),
    "cc_chunk_table_fill": (C.c_int64, [C.POINTER(C.c_uint64), C.c_int32, C.c_int32, C.POINTER(C.c_uint32), C.c_int64]),
    "cc_ordered_table_fill": (C.c_int64, [C.POINTER(C.c_uint64), C.c_int32, C.c_int32, C.POINTER(C.c_uint32), C.c_int64,
                                          C.POINTER(C.c_int64)]),
    "cc_default_chunk_elems": (C.c_int32, []),
    "cc_plan_create": (C.c_int, [C.POINTER(cc_tensor), C.c_int32, C.c_int32, C.c_int32, C.POINTER(C.c_void_p)]),
    "cc_plan_create_ex": (C.c_int, [C.POINTER(cc_tensor), C.c_int32, C.c_int32, C.c_int32, C.c_int32, C.POINTER(C.c_void_p)]),
    "cc_plan_destroy": (C.c_int, [C.c_void_p]),
    "cc_plan_set_schedule": (C.c_int, [C.c_void_p, C.c_int32, C.c_int32]),
    "cc_plan_schedule": (C.c_int, [C.c_void_p, C.POINTER(C.c_int32), C.POINTER(C.c_int32)]),
    "cc_plan_set_chunk_elems": (C.c_int, [C.c_void_p, C.c_int32]),
    "cc_plan_layout": (C.c_int, [C.c_void_p, C.POINTER(C.c_int32), C.POINTER(C.c_int32), C.POINTER(C.c_int32)]),
    "cc_plan_set_cache_policy": (C.c_int, [C.c_void_p, C.c_int32]),
    "cc_plan_reserve_unfused": (C.c_int, [C.c_void_p]),
    "cc_plan_set_meeting_limit": (C.c_int, [C.c_void_p, C.c_int32]),
    "cc_plan_queue_state": (C.c_int, [C.c_void_p, C.POINTER(C.c_uint32), C.POINTER(C.c_uint64), C.c_void_p]),
    "cc_plan_autotune": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_int32, C.c_void_p, C.c_void_p,
                                   C.POINTER(C.c_float), C.POINTER(C.c_float)]),
    "cc_plan_info": (C.c_int, [C.c_void_p, C.POINTER(C.c_uint64), C.POINTER(C.c_int64), C.POINTER(C.c_uint64)]),
    "cc_fused_adam_step": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p]),
    "cc_fused_adam_step_static": (C.c_int, [C.POINTER(cc_tensor), C.c_int32, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p]),
    "cc_fused_lamb_step": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p]),
    "cc_fused_lamb_phase1": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p]),
    "cc_fused_lamb_phase2": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p]),
    "cc_lamb_norm_buffer": (C.c_int, [C.c_void_p, C.POINTER(C.c_void_p)]),
    "cc_lamb_norms_read": (C.c_int, [C.c_void_p, C.POINTER(C.c_double), C.c_void_p]),
    "cc_unfused_adam_step": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p]),
    "cc_unfused_adam_step_ex": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p, C.c_int32]),
    "cc_unfused_lamb_step": (C.c_int, [C.c_void_p, C.POINTER(cc_hparams), C.c_void_p, C.c_void_p]),
    "cc_fused_epilogue": (C.c_int, [C.POINTER(cc_epilogue), C.c_void_p]),
    "cc_unfused_epilogue": (C.c_int, [C.POINTER(cc_epilogue), C.c_void_p, C.c_void_p]),
    "cc_pattern_probe": (C.c_int, [C.POINTER(cc_tensor), C.c_int32, C.c_int32, C.c_int32, C.c_void_p, C.c_void_p]),
    "cc_copy_probe": (C.c_int, [C.c_void_p, C.c_void_p, C.c_uint64, C.c_void_p]),
    "cc_device_info": (C.c_int, [C.POINTER(C.c_int32), C.POINTER(C.c_int32), C.POINTER(C.c_int32), C.POINTER(C.c_uint64)]),
    "cc_last_error": (C.c_char_p, []),
    "cc_version": (C.c_int, []),
}


def load():
    """Loads libccfused.so (built by paper_2105_05720_amd.build) and types its entry points."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(
                "%s is missing: build it with `python -m paper_2105_05720_amd.build` (there is no CPU fallback)" % LIB_PATH)
        lib = C.CDLL(LIB_PATH)
        for name, (res, args) in EXPORTS.items():
            fn = getattr(lib, name)          # AttributeError if the library does not export it
            fn.restype = res
            fn.argtypes = args
            if name.startswith(("cc_fused_", "cc_unfused_")):
                _at[name] = C.cast(fn, C.c_void_p).value
                as_bytes = [C.c_char_p if a in (C.POINTER(cc_hparams), C.POINTER(cc_tensor), C.POINTER(cc_epilogue)) else a for a in args]
                _packed[name] = C.CFUNCTYPE(res, *as_bytes)((name, lib))
        _lib = lib
    return _lib


def _check(rc: int) -> int:
    if rc < 0:
        raise CcError(int(rc), load().cc_last_error().decode())
    return rc


def _ptr(x) -> Optional[int]:
    if type(x) is int:
        return x
    try:
        return x.data_ptr()
    except AttributeError:
        return None if x is None else int(x)


_torch = _raw_stream = None


def _current_stream() -> Optional[int]:
    """The current stream's handle, without a Stream object around it (a torch Stream costs more than the rest of the call)."""
    global _torch, _raw_stream
    if _torch is None:
        import torch
        _raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
        _bind_native(torch)
        _torch = torch                    # last: where that raised (no device, say), the next call starts here again
    if _raw_stream is None:
        return _torch.cuda.current_stream().cuda_stream or None
    return _raw_stream(_torch.cuda.current_device()) or None


def _stream(stream) -> Optional[int]:
    if stream is None:
        return _current_stream()
    if hasattr(stream, "cuda_stream"):
        return stream.cuda_stream or None
    return int(stream) or None


@dataclass
class Tensor:
    """Python-side spelling of cc_tensor: torch tensors or integer device addresses."""
    numel: int
    w_in: object
    m_in: object
    v_in: object
    w_out: object
    m_out: object
    v_out: object
    w16_out: object
    grad: Sequence[object]
    weight_decay: float = 0.0


@dataclass
class Hyper:
    """Python-side spelling of cc_hparams."""
    lr: float = 1e-3
    beta1: float = 0.9
    beta2: float = 0.999
    eps: float = 1e-6
    loss_scale: float = 1.0
    step: int = 1
    grad_average: int = 0
    adam_mode: int = 1
    skip_mode: int = 0

    def to_c(self) -> cc_hparams:
        return cc_hparams(self.lr, self.beta1, self.beta2, self.eps, self.loss_scale, self.step,
                          self.grad_average, self.adam_mode, self.skip_mode)


def _hp(hp) -> cc_hparams:
    return hp if isinstance(hp, cc_hparams) else hp.to_c()


class Plan:
    """Owns a cc_plan handle and keeps the buffers it points at alive."""

    def __init__(self, handle: int, keep):
        self.handle = handle
        self._keep = keep

    def destroy(self):
        if self.handle:
            load().cc_plan_destroy(self.handle)
            self.handle = None

    def __del__(self):
        try:
            self.destroy()
        except Exception:
            pass


# ---- host helpers of the chunk table ----

def cc_default_chunk_elems() -> int:
    return load().cc_default_chunk_elems()


def cc_chunk_count(numels: Sequence[int], chunk_elems: int = 0) -> int:
    arr = (C.c_uint64 * max(len(numels), 1))(*numels)
    return _check(load().cc_chunk_count(arr, len(numels), chunk_elems))


def cc_chunk_table_fill(numels: Sequence[int], chunk_elems: int = 0, capacity: Optional[int] = None):
    n = cc_chunk_count(numels, chunk_elems) if capacity is None else capacity
    arr = (C.c_uint64 * max(len(numels), 1))(*numels)
    table = (C.c_uint32 * max(2 * n, 2))()
    k = _check(load().cc_chunk_table_fill(arr, len(numels), chunk_elems, table, n))
    return [(table[2 * i], table[2 * i + 1]) for i in range(k)]


def cc_ordered_table_fill(numels: Sequence[int], chunk_elems: int = 0):
    """([(tensor, chunk)] in the ordered schedule's order, number of full chunks)."""
    n = cc_chunk_count(numels, chunk_elems)
    arr = (C.c_uint64 * max(len(numels), 1))(*numels)
    table = (C.c_uint32 * max(2 * n, 2))()
    nfull = C.c_int64()
    k = _check(load().cc_ordered_table_fill(arr, len(numels), chunk_elems, table, n, C.byref(nfull)))
    return [(table[2 * i], table[2 * i + 1]) for i in range(k)], nfull.value


# ---- plan ----

def cc_plan_create(tensors: Sequence[Tensor], R: int, chunk_elems: int = 0) -> Plan:
    return cc_plan_create_ex(tensors, R, chunk_elems, CC_GRAD_F16)


def cc_plan_create_ex(tensors: Sequence[Tensor], R: int, chunk_elems: int = 0, grad_dtype: int = CC_GRAD_F16) -> Plan:
    arr = (cc_tensor * max(len(tensors), 1))()
    for i, t in enumerate(tensors):
        arr[i] = _c_tensor(t)
    handle = C.c_void_p()
    _check(load().cc_plan_create_ex(arr, len(tensors), R, chunk_elems, grad_dtype, C.byref(handle)))
    return Plan(handle.value, list(tensors))


def cc_plan_destroy(plan: Plan) -> None:
    plan.destroy()


def cc_plan_set_schedule(plan: Plan, schedule: int = CC_SCHEDULE_AUTO, workgroups: int = 0) -> None:
    _check(load().cc_plan_set_schedule(plan.handle, schedule, workgroups))


def cc_plan_schedule(plan: Plan):
    """(schedule the plan will use: CC_SCHEDULE_ORDERED or CC_SCHEDULE_PER_CHUNK, workgroups per launch)."""
    sched, wgs = C.c_int32(), C.c_int32()
    _check(load().cc_plan_schedule(plan.handle, C.byref(sched), C.byref(wgs)))
    return sched.value, wgs.value


def cc_plan_set_chunk_elems(plan: Plan, chunk_elems: int = 0) -> None:
    _check(load().cc_plan_set_chunk_elems(plan.handle, chunk_elems))


def cc_plan_layout(plan: Plan):
    """(chunk size in elements, threads per workgroup, CC_CACHE_STREAMING, CC_CACHE_RESIDENT or CC_CACHE_WRITE_THROUGH) the plan will use."""
    ce, blk, pol = C.c_int32(), C.c_int32(), C.c_int32()
    _check(load().cc_plan_layout(plan.handle, C.byref(ce), C.byref(blk), C.byref(pol)))
    return ce.value, blk.value, pol.value


def cc_plan_set_cache_policy(plan: Plan, policy: int = CC_CACHE_AUTO) -> None:
    _check(load().cc_plan_set_cache_policy(plan.handle, policy))


def cc_plan_reserve_unfused(plan: Plan) -> None:
    _check(load().cc_plan_reserve_unfused(plan.handle))


def cc_plan_set_meeting_limit(plan: Plan, polls: int) -> None:
    _check(load().cc_plan_set_meeting_limit(plan.handle, polls))


def cc_plan_queue_state(plan: Plan, stream=None):
    """(ticket counter, finished-workgroup word) of the ordered schedule after waiting for the stream; both 0 between launches."""
    nxt, done = C.c_uint32(), C.c_uint64()
    _check(load().cc_plan_queue_state(plan.handle, C.byref(nxt), C.byref(done), _stream(stream)))
    return nxt.value, done.value


def cc_plan_autotune(plan: Plan, hp, flag, optimizer: int = 0, stream=None):
    """Times the candidate layouts and schedules on the plan's own buffers and keeps the fastest.  Returns (ms per step
    of what was kept, ms per step with one workgroup per chunk under the layout the plan had)."""
    c = _hp(hp)
    best, per_chunk = C.c_float(), C.c_float()
    _check(load().cc_plan_autotune(plan.handle, C.byref(c), optimizer, _ptr(flag), _stream(stream), C.byref(best), C.byref(per_chunk)))
    return best.value, per_chunk.value


def cc_plan_info(plan: Plan):
    numel, chunks, tb = C.c_uint64(), C.c_int64(), C.c_uint64()
    _check(load().cc_plan_info(plan.handle, C.byref(numel), C.byref(chunks), C.byref(tb)))
    return numel.value, chunks.value, tb.value


# ---- steps ----

# A small shard's step costs the host more than the device, so the step calls go through the extension module (step_calls.cpp),
# which reads the objects' fields itself, from their second call on (the first one finds torch).  us per eager pass of a training
# loop that makes a new Hyper each time, packed bytes through ctypes / this: 6.1 / 5.1 for Adam on 4099 elements, R = 4; 6.9 / 5.4 for the
# static call on 100003, R = 2, and 8.0 / 6.3 on 200001, R = 16; 6.1 / 5.3 for LAMB on 10007; 5.7 / 4.6 for the epilogue on 21744, R = 4.
# What the module does not take (an integer address among a tensor's buffers, a stream that is given, a value out of its field's
# range, a wrong type) is packed into bytes in one go (native sizes and alignment, as in cc_hparams, cc_tensor and cc_epilogue).
# What does not pack goes through the ctypes structures, whose conversions and errors are the definition; so does a
# hyper-parameter object that is not exactly a Hyper, because its to_c() is what counts.
_PACK_HP = struct.Struct("5f4i").pack
_PACK_TENSOR = struct.Struct("Q7Q16Qf4x").pack
_PACK_EPILOGUE = struct.Struct("QQIi16QQQQf4xQ").pack
_NO_PTRS = (0,) * CC_MAX_R


def _hp_bytes(hp) -> bytes:
    if type(hp) is not Hyper:                 # a cc_hparams, or something that says with to_c() what it stands for
        return bytes(_hp(hp))
    try:
        return _PACK_HP(hp.lr, hp.beta1, hp.beta2, hp.eps, hp.loss_scale, hp.step, hp.grad_average, hp.adam_mode, hp.skip_mode)
    except (struct.error, OverflowError, TypeError):
        return bytes(_hp(hp))


def _ptrs(tensors) -> tuple:
    p = [x.data_ptr() for x in tensors[:CC_MAX_R]]
    return (*p, *_NO_PTRS[len(p):])


def _tensor_bytes(t: Tensor) -> bytes:
    try:
        return _PACK_TENSOR(t.numel, t.w_in.data_ptr(), t.m_in.data_ptr(), t.v_in.data_ptr(), t.w_out.data_ptr(),
                            t.m_out.data_ptr(), t.v_out.data_ptr(), t.w16_out.data_ptr(), *_ptrs(t.grad), t.weight_decay)
    except (struct.error, OverflowError, TypeError, AttributeError):
        return bytes(_c_tensor(t))


def _fn(name: str):
    if _lib is None:
        load()
    return _packed[name]


def _not_taken(*args) -> int:
    return 1


_native_step = _native_static = _native_epilogue = _not_taken


def _bind_native(torch=None) -> None:
    """Lets the step calls go through the extension module: torch is there, and its device has been looked at."""
    global _native_step, _native_static, _native_epilogue
    if _raw_stream is None:
        return
    try:
        from . import _step_calls as native
    except ImportError as e:              # not built, or for another Python: the packed bytes do as well
        warnings.warn("step calls go through ctypes, 1 to 2 us slower each: %s (python -m paper_2105_05720_amd.build)" % e, RuntimeWarning, stacklevel=2)
        return
    torch = torch or _torch
    torch.cuda.current_device()
    if native.bind(Plan, Hyper, Tensor, torch.Tensor, torch.nn.Parameter, torch._C._cuda_getDevice, _raw_stream):
        _native_step, _native_static, _native_epilogue = native.step, native.static_step, native.epilogue


def _unbind_native() -> None:
    """In a forked child torch's own calls say that it may not use the GPU."""
    global _native_step, _native_static, _native_epilogue
    _native_step = _native_static = _native_epilogue = _not_taken


os.register_at_fork(after_in_child=_unbind_native)


def _step(rc: int, name: str, plan: Plan, hp, flag, stream) -> None:
    """A step call that the extension module has not taken (rc = 1), or that has failed."""
    _check(rc if rc < 0 else _fn(name)(plan.handle, _hp_bytes(hp), _ptr(flag), _stream(stream)))


def cc_fused_adam_step(plan: Plan, hp, flag, stream=None) -> None:
    rc = _native_step(_at.get("cc_fused_adam_step"), plan, hp, flag, stream)
    if rc:
        _step(rc, "cc_fused_adam_step", plan, hp, flag, stream)


def cc_fused_adam_step_static(tensor: Tensor, R: int, hp, flag, stream=None) -> None:
    rc = _native_static(_at.get("cc_fused_adam_step_static"), tensor, R, hp, flag, stream)
    if rc:
        _check(rc if rc < 0 else _fn("cc_fused_adam_step_static")(_tensor_bytes(tensor), R, _hp_bytes(hp), _ptr(flag), _stream(stream)))


def cc_fused_lamb_step(plan: Plan, hp, flag, stream=None) -> None:
    rc = _native_step(_at.get("cc_fused_lamb_step"), plan, hp, flag, stream)
    if rc:
        _step(rc, "cc_fused_lamb_step", plan, hp, flag, stream)


def cc_fused_lamb_phase1(plan: Plan, hp, flag, stream=None) -> None:
    rc = _native_step(_at.get("cc_fused_lamb_phase1"), plan, hp, flag, stream)
    if rc:
        _step(rc, "cc_fused_lamb_phase1", plan, hp, flag, stream)


def cc_fused_lamb_phase2(plan: Plan, hp, flag, stream=None) -> None:
    rc = _native_step(_at.get("cc_fused_lamb_phase2"), plan, hp, flag, stream)
    if rc:
        _step(rc, "cc_fused_lamb_phase2", plan, hp, flag, stream)


def cc_unfused_adam_step(plan: Plan, hp, flag, stream=None) -> None:
    rc = _native_step(_at.get("cc_unfused_adam_step"), plan, hp, flag, stream)
    if rc:
        _step(rc, "cc_unfused_adam_step", plan, hp, flag, stream)


def cc_unfused_adam_step_ex(plan: Plan, hp, flag, stream=None, sum_dtype: int = CC_GRAD_F32) -> None:
    _check(_fn("cc_unfused_adam_step_ex")(plan.handle, _hp_bytes(hp), _ptr(flag), _stream(stream), sum_dtype))


def cc_unfused_lamb_step(plan: Plan, hp, flag, stream=None) -> None:
    rc = _native_step(_at.get("cc_unfused_lamb_step"), plan, hp, flag, stream)
    if rc:
        _step(rc, "cc_unfused_lamb_step", plan, hp, flag, stream)


def cc_lamb_norm_buffer(plan: Plan) -> int:
    p = C.c_void_p()
    _check(load().cc_lamb_norm_buffer(plan.handle, C.byref(p)))
    return p.value


def cc_lamb_norms_read(plan: Plan, T: int, stream=None):
    """Returns [(sum w^2, sum u^2)] per tensor after waiting for the stream."""
    buf = (C.c_double * max(2 * T, 2))()
    _check(load().cc_lamb_norms_read(plan.handle, buf, _stream(stream)))
    return [(buf[2 * i], buf[2 * i + 1]) for i in range(T)]


def _epilogue(partials, bias, residual, out, first: int, hidden: int, dropout_p: float, seed: int, numel=None) -> cc_epilogue:
    e = cc_epilogue()
    e.numel = residual.numel() if numel is None else numel
    e.first, e.hidden, e.R = first, hidden, len(partials)
    for r, x in enumerate(partials[:CC_MAX_R]):
        e.partial[r] = _ptr(x)
    e.bias, e.residual, e.out = _ptr(bias), _ptr(residual), _ptr(out)
    e.dropout_p, e.seed = dropout_p, seed
    return e


def _epilogue_bytes(partials, bias, residual, out, first, hidden, dropout_p, seed, numel) -> bytes:
    try:
        return _PACK_EPILOGUE(residual.numel() if numel is None else numel, first, hidden, len(partials), *_ptrs(partials),
                              bias.data_ptr(), residual.data_ptr(), out.data_ptr(), dropout_p, seed)
    except (struct.error, OverflowError, TypeError, AttributeError):
        return bytes(_epilogue(partials, bias, residual, out, first, hidden, dropout_p, seed, numel))


def cc_fused_epilogue(partials, bias, residual, out, first: int, hidden: int, dropout_p: float, seed: int, stream=None,
                      numel=None) -> None:
    rc = _native_epilogue(_at.get("cc_fused_epilogue"), partials, bias, residual, out, first, hidden, dropout_p, seed, stream, numel)
    if rc:
        _check(rc if rc < 0 else _fn("cc_fused_epilogue")(_epilogue_bytes(partials, bias, residual, out, first, hidden, dropout_p, seed, numel), _stream(stream)))


def cc_unfused_epilogue(partials, bias, residual, out, sum_scratch, first: int, hidden: int, dropout_p: float, seed: int,
                        stream=None, numel=None) -> None:
    e = _epilogue_bytes(partials, bias, residual, out, first, hidden, dropout_p, seed, numel)
    _check(_fn("cc_unfused_epilogue")(e, _ptr(sum_scratch), _stream(stream)))


def _c_tensor(t: Tensor) -> cc_tensor:
    c = cc_tensor()
    c.numel = t.numel
    c.w_in, c.m_in, c.v_in = _ptr(t.w_in), _ptr(t.m_in), _ptr(t.v_in)
    c.w_out, c.m_out, c.v_out = _ptr(t.w_out), _ptr(t.m_out), _ptr(t.v_out)
    c.w16_out = _ptr(t.w16_out)
    for r, g in enumerate(t.grad[:CC_MAX_R]):
        c.grad[r] = _ptr(g)
    c.weight_decay = t.weight_decay
    return c


def cc_pattern_probe(tensor: Tensor, R: int, what: int, cache_policy: int, sink, stream=None) -> None:
    c = _c_tensor(tensor)
    _check(load().cc_pattern_probe(C.byref(c), R, what, cache_policy, _ptr(sink), _stream(stream)))


def cc_copy_probe(dst, src, nbytes: int, stream=None) -> None:
    _check(load().cc_copy_probe(_ptr(dst), _ptr(src), nbytes, _stream(stream)))


def cc_device_info():
    """(compute units, memory clock kHz, memory bus bits, total bytes) of the current device."""
    cus, clk, bus, tot = C.c_int32(), C.c_int32(), C.c_int32(), C.c_uint64()
    _check(load().cc_device_info(C.byref(cus), C.byref(clk), C.byref(bus), C.byref(tot)))
    return cus.value, clk.value, bus.value, tot.value


def cc_last_error() -> str:
    return load().cc_last_error().decode()


def cc_version() -> int:
    return load().cc_version()

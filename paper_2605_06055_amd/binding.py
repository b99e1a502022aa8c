"""Binding of libmoe_rbf.so (argument marshalling only): native code for the usual arguments (_marshal), ctypes for the rest."""
from __future__ import annotations

import ctypes
import os
import sys
from typing import Optional

MOE_DTYPE_BF16, MOE_DTYPE_F32 = 0, 1
MOE_SCHEDULE_AUTO, MOE_SCHEDULE_PREFILL, MOE_SCHEDULE_DECODE = 0, 1, 2

_PKG = os.path.dirname(os.path.abspath(__file__))
_lib = None
_native = None          # the _marshal module, where it can be used


class MoeError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        detail = f" [{load_library().moe_last_launch_error().decode()}]" if code == -6 else ""
        super().__init__(f"{where}: {moe_strerror(code)} ({code}){detail}")


class MoeShape(ctypes.Structure):
    """Mirror of ``moe_shape``."""
    _fields_ = [("T", ctypes.c_int32), ("H", ctypes.c_int32), ("k", ctypes.c_int32), ("E", ctypes.c_int32),
                ("R", ctypes.c_int32), ("dtype", ctypes.c_int32), ("schedule", ctypes.c_int32),
                ("rank_id", ctypes.c_int32), ("region_stride_rows", ctypes.c_int64)]


class _PlanStruct(ctypes.Structure):
    """Mirror of ``moe_plan_t``."""
    _fields_ = [("expert_count", ctypes.c_void_p), ("rank_count", ctypes.c_void_p),
                ("expert_offset", ctypes.c_void_p), ("region_base", ctypes.c_void_p),
                ("send_idx", ctypes.c_void_p), ("row_map", ctypes.c_void_p), ("status", ctypes.c_void_p),
                ("workspace", ctypes.c_void_p), ("workspace_bytes", ctypes.c_size_t),
                ("source_count", ctypes.c_void_p), ("recv_count", ctypes.c_void_p), ("recv_offset", ctypes.c_void_p),
                ("dispatch_order", ctypes.c_void_p), ("prefetch", ctypes.c_void_p),
                ("prefetch_bytes", ctypes.c_size_t)]


def library_path() -> str:
    return os.environ.get("MOE_RBF_LIB", os.path.join(_PKG, "libmoe_rbf.so"))


def _bind_hip_runtime() -> None:
    """libmoe_rbf.so needs the HIP runtime by soname.  PyTorch ships its own libamdhip64 (same soname, not
    /opt/rocm's file); if the library were opened first it would pull in /opt/rocm's copy and torch
    would then load a second runtime whose streams and devices are not the library's.  Loading torch's
    copy first makes the dynamic loader reuse it for the library: one runtime per process."""
    try:
        import torch
        cand = os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so")
    except ImportError:
        cand = ""
    if os.path.exists(cand):
        ctypes.CDLL(cand, mode=ctypes.RTLD_GLOBAL)


def load_library():
    """Loads the built HIP library; raises if it has not been built (there is no fallback)."""
    global _lib
    if _lib is None:
        path = library_path()
        if not os.path.exists(path):
            raise ImportError(f"{path} not found: build it with `python -m paper_2605_06055_amd.build` "
                              "(or __graft_entry__.build()); this package has no CPU fallback")
        _bind_hip_runtime()
        lib = ctypes.CDLL(path)
        vp, i32p = ctypes.c_void_p, ctypes.POINTER(ctypes.c_int32)
        shp, plp = ctypes.POINTER(MoeShape), ctypes.POINTER(_PlanStruct)
        lib.moe_workspace_bytes.argtypes = [shp, ctypes.POINTER(ctypes.c_size_t)]
        lib.moe_window_rows.argtypes = [shp, ctypes.POINTER(ctypes.c_int64)]
        lib.moe_resolve_schedule.argtypes = [shp, i32p]
        lib.moe_plan.argtypes = [shp, vp, plp, vp]
        lib.moe_plan_static.argtypes = [shp, vp, plp, vp]
        lib.moe_dispatch.argtypes = [shp, vp, vp, plp, vp, vp]
        lib.moe_combine.argtypes = [shp, vp, vp, plp, vp, vp]
        lib.moe_dispatch_quant.argtypes = [shp, vp, vp, plp, vp, vp, vp]
        lib.moe_strerror.argtypes = [ctypes.c_int]
        lib.moe_strerror.restype = ctypes.c_char_p
        lib.moe_last_launch_error.argtypes = []
        lib.moe_last_launch_error.restype = ctypes.c_char_p
        for f in ("moe_workspace_bytes", "moe_window_rows", "moe_resolve_schedule", "moe_plan", "moe_plan_static",
                  "moe_dispatch",
                  "moe_dispatch_quant", "moe_combine"):
            getattr(lib, f).restype = ctypes.c_int
        _use_native(lib)
        _lib = lib
    return _lib


def _use_native(lib) -> None:
    """Hands the entry points to the native marshalling.  It reads torch tensors and Python objects by their layout: where it has not
    been built, or for another torch or Python, every call goes by way of ctypes."""
    global _native
    try:
        import torch                   # its libraries have to be loaded first
        from . import _marshal
    except ImportError:
        return
    if getattr(_marshal, "built_for", None) != _interpreter(torch):
        return
    at = [ctypes.cast(getattr(lib, f), ctypes.c_void_p).value
          for f in ("moe_plan", "moe_plan_static", "moe_dispatch", "moe_dispatch_quant", "moe_combine")]
    _marshal.use(*at, MoeShape, _PlanStruct, MoePlan, _raise)
    _native = _marshal


def _interpreter(torch) -> str:
    return f"torch {torch.__version__}, {sys.implementation.cache_tag}"


def _raise(code: int, where: str) -> None:
    raise MoeError(code, where)


def moe_strerror(code: int) -> str:
    return load_library().moe_strerror(code).decode()


def _check(code: int, where: str) -> None:
    if code != 0:
        raise MoeError(code, where)


def _ptr(t) -> Optional[int]:
    """Device pointer of a torch tensor (None stays NULL)."""
    if t is None or isinstance(t, int):
        return t
    assert t.is_contiguous(), "tensors must be dense row-major"
    return t.data_ptr()


_raw_stream = _device = _bad_fork = None


def _stream(stream) -> Optional[int]:
    """hipStream_t of a torch stream; None = the current stream of the current device."""
    if stream is None:
        if _raw_stream is None or _bad_fork():
            return _first_stream()
        return _raw_stream(_device())
    return stream if isinstance(stream, int) else stream.cuda_stream


def _first_stream() -> int:
    """The current stream by way of a torch.cuda.Stream, which initialises the device where that has not happened; later
    calls read the handle itself (torch.cuda.current_stream() builds two Python objects, about 2 us)."""
    global _raw_stream, _device, _bad_fork
    import torch
    handle = torch.cuda.current_stream().cuda_stream
    names = ("_cuda_getCurrentRawStream", "_cuda_getDevice", "_cuda_isInBadFork")
    if all(hasattr(torch._C, n) for n in names):
        raw, _device, _bad_fork = (getattr(torch._C, n) for n in names)
        if _native is not None:
            _native.streams(raw, _device, _bad_fork)
        _raw_stream = raw                       # set last: other threads test this one
    return handle


def moe_workspace_bytes(shape: MoeShape) -> int:
    out = ctypes.c_size_t(0)
    _check(load_library().moe_workspace_bytes(ctypes.byref(shape), ctypes.byref(out)), "moe_workspace_bytes")
    return out.value


def moe_window_rows(shape: MoeShape) -> int:
    out = ctypes.c_int64(0)
    _check(load_library().moe_window_rows(ctypes.byref(shape), ctypes.byref(out)), "moe_window_rows")
    return out.value


def moe_resolve_schedule(shape: MoeShape) -> int:
    out = ctypes.c_int32(0)
    _check(load_library().moe_resolve_schedule(ctypes.byref(shape), ctypes.byref(out)), "moe_resolve_schedule")
    return out.value


class MoePlan:
    """Device buffers of ``moe_plan_t`` held as torch tensors (memory plumbing only).  ``with_order=False`` leaves out the
    order list that only the unquantised prefill dispatch reads."""

    def __init__(self, shape: MoeShape, device="cuda", with_send_idx: bool = True, source_count=None,
                 with_order: bool = True):
        import torch
        N = shape.T * shape.k
        i32 = dict(dtype=torch.int32, device=device)
        self.expert_count = torch.empty(shape.E, **i32)
        self.rank_count = torch.empty(shape.R, **i32)
        self.expert_offset = torch.empty(shape.E + 1, **i32)
        self.region_base = torch.empty(shape.R + 1, **i32)
        self.send_idx = torch.empty(max(N, 1), **i32) if with_send_idx else None
        self.row_map = torch.empty(max(N, 1), **i32)
        self.status = torch.empty(4, **i32)
        self.workspace = torch.empty(moe_workspace_bytes(shape), dtype=torch.uint8, device=device)
        self.source_count = source_count          # [R,E] int32 counts of the other source ranks, or None
        self.recv_count = torch.empty(shape.E, **i32)
        self.recv_offset = torch.empty(shape.E + 1, **i32)
        self.dispatch_order = torch.empty(2 * max(N, 1), **i32) if with_order else None
        self.prefetch = None                      # tensor that moe_plan should pull into the caches (normally x), or None

    def struct(self) -> _PlanStruct:
        return _PlanStruct(_ptr(self.expert_count), _ptr(self.rank_count), _ptr(self.expert_offset),
                           _ptr(self.region_base), _ptr(self.send_idx), _ptr(self.row_map), _ptr(self.status),
                           _ptr(self.workspace), self.workspace.numel(), _ptr(self.source_count),
                           _ptr(self.recv_count), _ptr(self.recv_offset), _ptr(self.dispatch_order),
                           _ptr(self.prefetch),
                           0 if self.prefetch is None else self.prefetch.numel() * self.prefetch.element_size())


def _plan_struct(plan) -> _PlanStruct:
    return plan.struct() if isinstance(plan, MoePlan) else plan


def _slow(name: str, shape, before, plan, after, stream) -> int:
    """A call by way of ctypes: before the library is loaded and for arguments that the native marshalling does not read (it then
    returns None), with ctypes' conversions and errors."""
    lib = load_library()
    return getattr(lib, name)(shape, *map(_ptr, before), _plan_struct(plan), *map(_ptr, after), _stream(stream))


def moe_plan(shape: MoeShape, topk_idx, plan, stream=None) -> None:
    code = _native.plan(shape, topk_idx, plan, stream) if _native else None
    if code is None:
        code = _slow("moe_plan", shape, (topk_idx,), plan, (), stream)
    if code:
        raise MoeError(code, "moe_plan")


def moe_plan_static(shape: MoeShape, topk_idx, plan, stream=None) -> None:
    code = _native.plan_static(shape, topk_idx, plan, stream) if _native else None
    if code is None:
        code = _slow("moe_plan_static", shape, (topk_idx,), plan, (), stream)
    if code:
        raise MoeError(code, "moe_plan_static")


def moe_dispatch(shape: MoeShape, x, topk_idx, plan, window, stream=None) -> None:
    code = _native.dispatch(shape, x, topk_idx, plan, window, stream) if _native else None
    if code is None:
        code = _slow("moe_dispatch", shape, (x, topk_idx), plan, (window,), stream)
    if code:
        raise MoeError(code, "moe_dispatch")


def moe_dispatch_quant(shape: MoeShape, x, topk_idx, plan, window_q, window_scale, stream=None) -> None:
    code = _native.dispatch_quant(shape, x, topk_idx, plan, window_q, window_scale, stream) if _native else None
    if code is None:
        code = _slow("moe_dispatch_quant", shape, (x, topk_idx), plan, (window_q, window_scale), stream)
    if code:
        raise MoeError(code, "moe_dispatch_quant")


def moe_combine(shape: MoeShape, expert_out, topk_w, plan, y, stream=None) -> None:
    code = _native.combine(shape, expert_out, topk_w, plan, y, stream) if _native else None
    if code is None:
        code = _slow("moe_combine", shape, (expert_out, topk_w), plan, (y,), stream)
    if code:
        raise MoeError(code, "moe_combine")


def _bind(shape, plan, prefill, x, topk_idx, topk_w, window, expert_out, y, stream, buffers):
    """A layer's two calls on fixed addresses, (dispatch, combine): natively, or by way of ctypes for what the native marshalling
    does not read (it then returns None).  Each of the two keeps `buffers`, the owners of the memory."""
    lib = load_library()
    calls = _native.bind(shape, plan, prefill, x, topk_idx, topk_w, window, expert_out, y, stream, buffers) if _native else None
    if calls is not None:
        return calls.dispatch, calls.combine
    vp = ctypes.c_void_p
    shape, plan = ctypes.byref(shape), ctypes.byref(plan)
    x, topk_idx, topk_w, window, expert_out, y, stream = map(vp, (x, topk_idx, topk_w, window, expert_out, y, stream))

    def dispatch():
        if prefill:
            _check(lib.moe_plan(shape, topk_idx, plan, stream), "moe_plan")
        _check(lib.moe_dispatch(shape, x, topk_idx, plan, window, stream), "moe_dispatch")

    def combine():
        _check(lib.moe_combine(shape, expert_out, topk_w, plan, y, stream), "moe_combine")

    dispatch.buffers = combine.buffers = buffers
    return dispatch, combine

"""Thin binding of libpipad.so: argument marshalling only, by ctypes and, for plain arguments of the calls that a
step makes, by _host (csrc/pipad_host.cpp), which hands anything else back to the code here.  Where that native half is not
there and cannot be built (no compiler, no headers) everything goes by ctypes, at 10 to 20 us more per step.

Every step of the path (overlap extraction, normalisation, aggregation) runs in the HIP kernels of
the library; nothing here computes.  PyTorch supplies device memory and streams.  There is no CPU
fallback: if the library cannot be loaded the import of this module's functions fails loudly.

The names mirror ``include/pipad.h``:
  pipad_frame_build_overlap  -> :func:`frame_build_overlap`   (Section 4.1 / 4.3: overlap + exclusive parts)
  pipad_frame_aggregate      -> :func:`frame_aggregate`       (Section 4.2: parallel + exclusive aggregation)
  pipad_frame_common / _delta / _dinv -> :meth:`Frame.common`, :meth:`Frame.delta`, :meth:`Frame.dinv`
"""
from __future__ import annotations

import ctypes
import functools
import importlib.util
import itertools
import os
import struct
import subprocess
import warnings
import weakref
from typing import List, Optional, Sequence, Tuple, Union

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libpipad.so")
MAX_K = 32
VALIDATE = 1

_lib = None
_host = None      # the native half of this module, or None
_address: dict = {}  # the library's functions for it


class PipadError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"libpipad: {text} (status {status})")
        self.status = status


class _Csr(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int32), ("nnz", ctypes.c_int32),
                ("rowptr", ctypes.c_void_p), ("colidx", ctypes.c_void_p)]


ALLOC_FN = ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)

# symbol -> (restype, argtypes); also the list the ABI test checks against include/pipad.h.  Arrays that a call
# only reads are plain pointers: packed bytes are made in a fraction of the time that a ctypes array takes (16
# descriptors 8.6 us, packed 0.8).
_vp, _i32, _i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
SIGNATURES = {
    "pipad_frame_build_overlap": (ctypes.c_int, [_i32, _i32, _vp, ctypes.c_uint32, _vp, _vp, _vp, ctypes.POINTER(_vp)]),
    "pipad_frame_common": (ctypes.c_int, [_vp, ctypes.POINTER(_Csr)]),
    "pipad_frame_delta": (ctypes.c_int, [_vp, _i32, ctypes.POINTER(_Csr)]),
    "pipad_frame_dinv": (ctypes.c_int, [_vp, ctypes.POINTER(_vp), ctypes.POINTER(_i64),
                                        ctypes.POINTER(_i64)]),
    "pipad_frame_shape": (ctypes.c_int, [_vp, ctypes.POINTER(_i32), ctypes.POINTER(_i32)]),
    "pipad_frame_aggregate": (ctypes.c_int, [_vp, _i32, _vp, _i64, _vp, _i64, _vp]),
    "pipad_frame_aggregate_subset": (ctypes.c_int, [_vp, _i32, _vp, _i32, _vp, _i64, _vp, _i64, _vp]),
    "pipad_frame_aggregate_static": (ctypes.c_int, [_vp, _i32, _vp, _i64, _vp, _i64, _vp]),
    "pipad_frame_aggregate_update": (ctypes.c_int, [_vp, _i32, _vp, _i64, _vp, _i64, _vp, _i32, _vp, _i64, _vp, _i64, _vp]),
    "pipad_frame_transpose": (ctypes.c_int, [_vp, _vp, _vp, _vp, ctypes.POINTER(_vp)]),
    "pipad_frame_temporaries": (ctypes.c_int, [_vp, ctypes.POINTER(_vp), ctypes.POINTER(ctypes.c_size_t)]),
    "pipad_recommended_row_stride": (ctypes.c_int64, [_i32]),
    "pipad_frame_destroy": (None, [_vp]),
    "pipad_strerror": (ctypes.c_char_p, [ctypes.c_int]),
    "pipad_last_hip_error": (ctypes.c_char_p, []),
    "pipad_set_option": (ctypes.c_int, [ctypes.c_char_p, _i64]),
    # include/pipad_ceilings.h (measurement kernels)
    "pipad_ceiling_stream_read": (ctypes.c_int, [_vp, ctypes.c_size_t, _vp, _vp]),
    "pipad_ceiling_stream_copy": (ctypes.c_int, [_vp, _vp, ctypes.c_size_t, _vp]),
    "pipad_ceiling_gather": (ctypes.c_int, [_vp, _i64, _i32, _i64, _vp, _i64, _i32, _vp, _vp]),
    "pipad_ceiling_sink_floats": (ctypes.c_size_t, []),
    "pipad_get_option": (ctypes.c_int, [ctypes.c_char_p, ctypes.POINTER(_i64)]),
}


# The packed forms of k snapshot descriptors and of k pointers.
_pack_csr = functools.lru_cache(64)(lambda k: struct.Struct("IIPP" * k).pack)  # (pipad_csr_t, sizes mod 2^32)
_pack_pointers = functools.lru_cache(64)(lambda k: struct.Struct(f"{k}P").pack)


def load_library():
    """Loads libpipad.so (building it first only if it does not exist yet).  The environment
    variable PIPAD_LIBRARY names another build of the library to load instead (measurement builds,
    see build.py); a missing file is an error, never a fallback."""
    global _lib, _host
    if _lib is None:
        _host = _load_host()
        path = os.environ.get("PIPAD_LIBRARY") or LIB_PATH
        if path == LIB_PATH and not os.path.exists(LIB_PATH):
            from . import build as _build
            _build.build()
        lib = ctypes.CDLL(path)
        for name, (res, args) in SIGNATURES.items():
            fn = getattr(lib, name)
            fn.restype = res
            fn.argtypes = args
            _address[name] = ctypes.cast(fn, _vp).value
        _lib = lib
    return _lib


def _load_host():
    """The native half of this module, built first where there is none for this interpreter and torch; None where that
    cannot be done."""
    from . import build as _build
    path = _build.host_path()
    try:
        if not os.path.exists(path):
            _build.build_host()
        spec = importlib.util.spec_from_file_location(f"{__package__}._host", path)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
        return module
    except (OSError, ImportError, subprocess.CalledProcessError) as why:
        warnings.warn(f"the binding's native half is not there, calls take longer without it: {why}", RuntimeWarning, stacklevel=3)
        return None


def _check(status: int) -> None:
    if status != 0:
        lib = load_library()
        text = lib.pipad_strerror(status).decode()
        if status == -5:
            text += ": " + lib.pipad_last_hip_error().decode()
        raise PipadError(status, text)


def set_option(key: str, value: int) -> None:
    _check(load_library().pipad_set_option(key.encode(), int(value)))


def get_option(key: str) -> int:
    v = _i64(0)
    _check(load_library().pipad_get_option(key.encode(), ctypes.byref(v)))
    return int(v.value)


class _DevArray:
    """Exposes a raw device pointer through __cuda_array_interface__ (view, copied at once by the caller)."""

    def __init__(self, ptr: int, count: int, typestr: str):
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": typestr,
                                         "data": (ptr, False), "version": 2}


def _copy_from_device(ptr: Optional[int], count: int, dtype: torch.dtype, device) -> torch.Tensor:
    if count == 0 or not ptr:
        return torch.empty(0, dtype=dtype, device=device)
    typestr = {torch.int32: "<i4", torch.float32: "<f4"}[dtype]
    return torch.as_tensor(_DevArray(ptr, count, typestr), device=device).clone()


_unused_size = ctypes.byref(ctypes.c_size_t())  # where calls put a size that nobody asks for

# The current stream of a device as a plain handle and the current device's index, without the
# objects that torch.cuda.current_stream() and torch.cuda.device() make on every call: on small
# frames the host side of a call takes longer than its kernels.
_current_raw_stream = torch._C._cuda_getCurrentRawStream
_current_device = torch._C._cuda_getDevice


def _on_device(index: int, fn, *args) -> int:
    """fn(*args) with the given device current."""
    if _current_device() == index:
        return fn(*args)
    with torch.cuda.device(index):
        return fn(*args)


def _device_index(device) -> int:
    return device.index if device.index is not None else torch.cuda.current_device()


Snapshot = Tuple[torch.Tensor, torch.Tensor]  # (rowptr int32[n+1], colidx int32[nnz]) on the GPU


class Frame:
    """Owner of one ``pipad_frame_t``.  Built by :func:`frame_build_overlap`."""

    def __init__(self, handle: int, n: int, k: int, device, buffers, key: Optional[int] = None,
                 stream=None):
        self._h = handle
        self.n, self.k, self.device = n, k, device
        self._index = index = _device_index(device)
        self._buffers = buffers  # what the library got through the allocator callback, by address
        # torch's allocator hands memory out, and takes it back, in the order of the stream that
        # was current at the allocation; work on any other stream has to be waited for in close().  Scratch
        # that a later call asks for is ordered by the stream that is current then, and the frame's own has to be
        # waited for as well from there on.
        self._alloc_stream = _current_raw_stream(index)
        self._other_streams = {}
        self._temp = None
        built_on = self._alloc_stream if stream is None else self._stream(stream)
        # (key: the memory is torch's.  In one piece it holds no temporaries of their own.)
        if key is not None and len(buffers) != 1:
            # the build's temporaries can go back to the allocator as soon as the build's kernels have
            # run: at once where its order is that of the build's stream, else behind an event
            ptr = _vp()
            _check(_lib.pipad_frame_temporaries(handle, ctypes.byref(ptr), _unused_size))
            if ptr.value:
                if built_on == self._alloc_stream:
                    self._buffers.pop(ptr.value, None)
                else:
                    event = torch.cuda.Event()
                    event.record(self._other_streams[built_on])
                    self._temp = (ptr.value, event)

    def _stream(self, stream) -> int:
        """Handle of the stream a call runs on; streams other than the allocator's are remembered."""
        current = _current_raw_stream(self._index)
        raw = int(stream.cuda_stream) if stream is not None else current
        if raw != self._alloc_stream and raw not in self._other_streams:
            self._other_streams[raw] = stream if stream is not None else torch.cuda.current_stream(self._index)
        if current != self._alloc_stream and self._alloc_stream not in self._other_streams:
            own = self._alloc_stream
            self._other_streams[own] = torch.cuda.ExternalStream(own, self.device) if own else torch.cuda.default_stream(self.device)
        return raw

    def _release_temporaries(self) -> None:
        if self._temp is not None and self._temp[1].query():
            self._buffers.pop(self._temp[0], None)
            self._temp = None

    def close(self) -> None:
        if self._h:
            # work of this frame may still be running on streams other than the one its buffers
            # are ordered on
            for s in self._other_streams.values():
                s.synchronize()
            load_library().pipad_frame_destroy(self._h)
            self._h = None
            self._temp = None
            self._buffers.clear()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _view(self, t: Optional[int]) -> Tuple[torch.Tensor, torch.Tensor]:
        lib = load_library()
        v = _Csr()
        if t is None:
            _check(lib.pipad_frame_common(self._h, ctypes.byref(v)))
        else:
            _check(lib.pipad_frame_delta(self._h, t, ctypes.byref(v)))
        torch.cuda.synchronize(self.device)
        rowptr = _copy_from_device(v.rowptr, self.n + 1, torch.int32, self.device)
        col = _copy_from_device(v.colidx, v.nnz, torch.int32, self.device)
        return rowptr, col

    def common(self) -> Snapshot:
        """Copy of the overlap CSR (pipad_frame_common)."""
        return self._view(None)

    def delta(self, t: int) -> Snapshot:
        """Copy of the exclusive CSR of snapshot t (pipad_frame_delta)."""
        return self._view(t)

    def dinv(self) -> torch.Tensor:
        """Copy of D^-1/2 as a float32[k, n] tensor (pipad_frame_dinv)."""
        lib = load_library()
        ptr, ldn, lds = _vp(), _i64(), _i64()
        _check(lib.pipad_frame_dinv(self._h, ctypes.byref(ptr), ctypes.byref(ldn), ctypes.byref(lds)))
        assert ldn.value == 1 and lds.value == self.n
        torch.cuda.synchronize(self.device)
        return _copy_from_device(ptr.value, self.k * self.n, torch.float32, self.device).view(self.k, self.n)


# Memory out of PyTorch's caching allocator without the native half.  One callback for all frames, which finds a frame's buffers by the
# key it is called with: a ctypes callback sits in a reference cycle, and with one per frame the garbage collector walked
# the whole program every few hundred frames.
_owners: "weakref.WeakValueDictionary[int, _Buffers]" = weakref.WeakValueDictionary()
_next_key = itertools.count(1).__next__


class _Buffers(dict):
    """The tensors handed out for a frame, by address, which keeps them alive."""

    def __init__(self, device):
        super().__init__()
        self._device, self._key = device, _next_key()
        _owners[self._key] = self

    def context(self) -> int:
        return self._key


def _allocate(nbytes, key):
    try:
        buffers = _owners[key]
        buf = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=buffers._device)
        buffers[buf.data_ptr()] = buf
        return buf.data_ptr()
    except Exception:  # out of memory -> NULL -> PIPAD_ERR_ALLOC
        return None


_allocate_callback = ALLOC_FN(_allocate)
_ALLOCATE = ctypes.cast(_allocate_callback, _vp).value


def _build(index: int, n: int, k: int, device, allocator: str, stream, fn, *args) -> Frame:
    """The frame that fn(*args, allocator, its context, stream, result) makes."""
    if allocator not in ("torch", "library"):
        raise ValueError("allocator must be 'torch' or 'library'")
    # (the library takes memory from PyTorch's caching allocator through a callback, which keeps it in `buffers`)
    buffers, callback, context = {}, None, None
    if allocator == "torch":
        buffers = _Buffers(device) if _host is None else _host.Buffers()
        callback, context = _ALLOCATE if _host is None else _host.ALLOCATE, buffers.context()
    out = _vp()
    raw = int(stream.cuda_stream) if stream is not None else _current_raw_stream(index)
    _check(_on_device(index, fn, *args, callback, context, raw, ctypes.byref(out)))
    return Frame(out.value, n, k, device, buffers, context, stream)


def frame_transpose(frame: Frame, allocator: str = "torch", stream=None) -> Frame:
    """pipad_frame_transpose: the frame of the transposed patterns with the same D^-1/2; aggregating
    with it applies the transposed operator (the backward pass for directed patterns)."""
    index = frame._index
    if _host is not None and allocator == "torch" and _current_device() == index:
        buffers = _host.Buffers()
        made = _host.transpose(_address["pipad_frame_transpose"], frame._h, buffers,
                               int(stream.cuda_stream) if stream is not None else _current_raw_stream(index))
        if made is not None:
            status, handle = made
            if status:
                _check(status)
            return Frame(handle, frame.n, frame.k, frame.device, buffers, 1, stream)
    return _build(index, frame.n, frame.k, frame.device, allocator, stream,
                  load_library().pipad_frame_transpose, frame._h)


def frame_build_overlap(snapshots: Sequence[Snapshot], validate: bool = False,
                        allocator: str = "torch", stream=None) -> Frame:
    """pipad_frame_build_overlap: k CSR snapshots -> frame (overlap CSR + k exclusive CSRs + D^-1/2).

    ``allocator="torch"`` hands every frame buffer out of PyTorch's caching allocator through the
    C callback; ``"library"`` lets the library hipMalloc its own."""
    lib = load_library()
    k = len(snapshots)
    if k < 1:
        raise ValueError("a frame needs at least one snapshot")
    rp0 = snapshots[0][0]
    n = rp0.numel() - 1
    device = rp0.device
    if not rp0.is_cuda:
        raise ValueError("snapshots must be contiguous int32 tensors on one GPU")
    index = _device_index(device)
    flags = VALIDATE if validate else 0
    if _host is not None and allocator == "torch" and _current_device() == index:
        buffers = _host.Buffers()
        made = _host.build(_address["pipad_frame_build_overlap"], snapshots, index, flags, buffers,
                           int(stream.cuda_stream) if stream is not None else _current_raw_stream(index))
        if made is not None:
            status, handle, n = made
            if status:
                _check(status)
            return Frame(handle, n, k, device, buffers, 1, stream)
    int32 = torch.int32
    descr = []
    for rp, col in snapshots:
        if rp.dtype is not int32 or rp.get_device() != index or not rp.is_contiguous() or \
                col.dtype is not int32 or col.get_device() != index or not col.is_contiguous():
            raise ValueError("snapshots must be contiguous int32 tensors on one GPU")
        nnz = col.numel()
        descr += (rp.numel() - 1 & 0xffffffff, nnz & 0xffffffff, rp.data_ptr(), col.data_ptr() if nnz else 0)
    return _build(index, n, k, device, allocator, stream, lib.pipad_frame_build_overlap,
                  n, k, _pack_csr(k)(*descr), flags)


Features = Union[torch.Tensor, Sequence[torch.Tensor]]


def _operand(x: Features, n: int, k: int, name: str) -> Tuple[List[int], int, int]:
    """Returns (k device pointers, row stride in elements, F).  Accepts a list of k [n, F] matrices
    sharing one row stride, or one [n, k, F] tensor (the physically concatenated coalescent operand)."""
    float32 = torch.float32
    if isinstance(x, torch.Tensor):
        shape = x.shape
        if len(shape) != 3 or shape[0] != n or shape[1] != k:
            raise ValueError(f"{name}: a single tensor must have shape [n, k, F]")
        if x.dtype is not float32 or not x.is_cuda:
            raise ValueError(f"{name}: every matrix must be float32 [n, F] on the GPU")
        F = shape[2]
        s0, s1, s2 = x.stride()
        if F > 1 and s2 != 1:
            raise ValueError(f"{name}: feature columns must be contiguous")
        first = x.data_ptr()
        return [first + 4 * s1 * t for t in range(k)], (s0 if n > 1 else max(s0, F)), F
    mats = list(x)
    if len(mats) != k:
        raise ValueError(f"{name}: need k = {k} matrices")
    shape = mats[0].shape
    F = shape[1]
    if len(shape) != 2 or shape[0] != n:
        raise ValueError(f"{name}: every matrix must be float32 [n, F] on the GPU")
    strides = mats[0].stride()
    if F > 1 and strides[1] != 1:
        raise ValueError(f"{name}: feature columns must be contiguous")
    ptrs = []
    for m in mats:
        if m.dtype is not float32 or not m.is_cuda or m.shape != shape:
            raise ValueError(f"{name}: every matrix must be float32 [n, F] on the GPU")
        if m.stride() != strides:
            if F > 1 and m.stride(1) != 1:
                raise ValueError(f"{name}: feature columns must be contiguous")
            if n > 1 and m.stride(0) != strides[0]:
                raise ValueError(f"{name}: all matrices must share one row stride")
        ptrs.append(m.data_ptr())
    return ptrs, (strides[0] if n > 1 else max(strides[0], F)), F


def frame_aggregate(frame: Frame, X: Features, Y: Optional[Features] = None, stream=None,
                    static_scratch: bool = False) -> Features:
    """pipad_frame_aggregate: Y_t = D_t^-1/2 (A_t + I) D_t^-1/2 X_t for every snapshot of the frame.

    Y is allocated like X when not given.  Only enqueues work on the stream.
    ``static_scratch=True`` calls pipad_frame_aggregate_static instead (no device allocation inside
    the library; pass Y, or this wrapper allocates it before the call)."""
    lib = load_library()
    n, k = frame.n, frame.k
    if _host is not None and Y is not None and _current_device() == frame._index:
        frame._release_temporaries()
        status = _host.aggregate(_address["pipad_frame_aggregate_static" if static_scratch else "pipad_frame_aggregate"],
                                 frame._h, n, k, X, Y, frame._stream(stream))
        if status is not None:
            if status:
                _check(status)
            return Y
    xp, ldx, F = _operand(X, n, k, "X")
    if Y is None:
        if isinstance(X, torch.Tensor):
            Y = torch.empty_like(X, memory_format=torch.contiguous_format)
        else:
            Y = [torch.empty((n, F), dtype=torch.float32, device=frame.device) for _ in range(k)]
    yp, ldy, Fy = _operand(Y, n, k, "Y")
    if Fy != F:
        raise ValueError("X and Y must have the same number of feature columns")
    pack = _pack_pointers(k)
    frame._release_temporaries()
    fn = lib.pipad_frame_aggregate_static if static_scratch else lib.pipad_frame_aggregate
    _check(_on_device(frame._index, fn, frame._h, F, pack(*xp), ldx, pack(*yp), ldy, frame._stream(stream)))
    return Y


def frame_aggregate_subset(frame: Frame, snapshots: Sequence[int], X: Sequence[Optional[torch.Tensor]],
                           Y: Sequence[Optional[torch.Tensor]], stream=None) -> None:
    """pipad_frame_aggregate_subset: Y[t] = D_t^-1/2 (A_t + I) D_t^-1/2 X[t] for the listed snapshots
    of the frame only (inter-frame reuse: the other Y_t are kept from the previous frame).  X and Y
    are lists of k entries; those of snapshots not listed may be None."""
    lib = load_library()
    n, k = frame.n, frame.k
    sel = [int(t) for t in snapshots]
    if not sel:
        return
    if len(X) != k or len(Y) != k:
        raise ValueError("X and Y must have k entries")
    if _host is not None and _current_device() == frame._index:
        frame._release_temporaries()
        status = _host.subset(_address["pipad_frame_aggregate_subset"], frame._h, n, k, sel, X, Y, frame._stream(stream))
        if status is not None:
            if status:
                _check(status)
            return
    F, ldx, ldy = None, None, None
    xa, ya = [0] * k, [0] * k
    for t in sel:
        for m, name in ((X[t], "X"), (Y[t], "Y")):
            if m is None or m.dtype != torch.float32 or not m.is_cuda or m.dim() != 2 or m.shape[0] != n:
                raise ValueError(f"{name}[{t}] must be a float32 [n, F] matrix on the GPU")
            if m.shape[1] > 1 and m.stride(1) != 1:
                raise ValueError("feature columns must be contiguous")
        if F is None:
            F = int(X[t].shape[1])
            ldx = int(X[t].stride(0)) if n > 1 else max(int(X[t].stride(0)), F)
            ldy = int(Y[t].stride(0)) if n > 1 else max(int(Y[t].stride(0)), F)
        if X[t].shape[1] != F or Y[t].shape[1] != F or (n > 1 and (X[t].stride(0) != ldx or Y[t].stride(0) != ldy)):
            raise ValueError("the chosen matrices must share their shape and row strides")
        xa[t], ya[t] = X[t].data_ptr(), Y[t].data_ptr()
    arr = (_i32 * len(sel))(*sel)
    pack = _pack_pointers(k)
    frame._release_temporaries()
    _check(_on_device(frame._index, lib.pipad_frame_aggregate_subset, frame._h, len(sel), arr, F, pack(*xa), ldx,
                      pack(*ya), ldy, frame._stream(stream)))


def frame_aggregate_update(frame: Frame, X: Features, W: torch.Tensor,
                           bias: Optional[torch.Tensor] = None, H: Optional[Features] = None,
                           A: Optional[Features] = None, stream=None) -> Features:
    """pipad_frame_aggregate_update: H_t = (D_t^-1/2 (A_t + I) D_t^-1/2 X_t) W + bias for every
    snapshot of the frame.  W is a float32 [F, Fo] device matrix (row stride >= Fo), bias a float32
    [Fo] device vector or None.  H is allocated (k matrices [n, Fo]) when not given; A, when given,
    receives the aggregation results.  Only enqueues work on the stream."""
    lib = load_library()
    n, k = frame.n, frame.k
    if _host is not None and H is not None and _current_device() == frame._index:
        frame._release_temporaries()
        status = _host.update(_address["pipad_frame_aggregate_update"], frame._h, n, k, X, W, bias, A, H, frame._stream(stream))
        if status is not None:
            if status:
                _check(status)
            return H
    xp, ldx, F = _operand(X, n, k, "X")
    if W.dtype != torch.float32 or W.dim() != 2 or W.shape[0] != F or W.stride(1) != 1:
        raise ValueError("W must be a float32 [F, Fo] matrix with unit column stride")
    Fo = int(W.shape[1])
    if bias is not None and (bias.dtype != torch.float32 or bias.dim() != 1 or
                             bias.shape[0] != Fo or bias.stride(0) != 1):
        raise ValueError("bias must be a contiguous float32 vector of Fo entries")
    if H is None:
        H = [torch.empty((n, Fo), dtype=torch.float32, device=frame.device) for _ in range(k)]
    hp, ldh, Fh = _operand(H, n, k, "H")
    if Fh != Fo:
        raise ValueError("H must have Fo feature columns")
    pack = _pack_pointers(k)
    xa, ha = pack(*xp), pack(*hp)
    aa, lda = None, F
    if A is not None:
        ap, lda, Fa = _operand(A, n, k, "A")
        if Fa != F:
            raise ValueError("A must have F feature columns")
        aa = pack(*ap)
    frame._release_temporaries()
    _check(_on_device(
        frame._index, lib.pipad_frame_aggregate_update,
        frame._h, F, xa, ldx, W.data_ptr(), W.stride(0) if F > 1 else max(Fo, W.stride(0)),
        bias.data_ptr() if bias is not None else None, Fo, aa, lda, ha, ldh, frame._stream(stream)))
    return H

"""Python binding of the BLCO sparse MTTKRP library (``libblco.so``, C ABI in include/blco.h).

Argument marshalling only: every step of the computation runs in the library's
HIP kernels.  PyTorch provides device memory and streams.  ``torch`` is
imported before the library is loaded so that the library binds to the HIP
runtime torch already uses (one runtime per process).

Method: Nguyen et al., "Efficient, Out-of-Memory Sparse MTTKRP on Massively
Parallel Architectures", ICS '22 — the BLCO format (Section 4) and its MTTKRP
(Section 5).
"""
from __future__ import annotations

import ctypes
import os

import numpy as np
import torch  # noqa: F401  (must precede loading libblco.so)

__all__ = ["BLCOTensor", "build", "mttkrp", "mttkrp_acc", "mttkrp_v", "mttkrp_stream",
           "mttkrp_stream_all", "sampled_loss", "cp_grad",
           "cast_bf16", "atomic_probe", "gather_probe", "CPLoss", "BLCOError", "lib", "library_path"]

_HERE = os.path.dirname(os.path.abspath(__file__))
_SO = os.path.join(_HERE, "libblco.so")
_lib = None

MAX_MODES = 8
F32, BF16 = 0, 1
PLACEMENTS = {"device": 0, "pinned": 1, "host": 2}
STATUS = {0: "OK", -1: "EINVAL", -2: "ENOMEM", -3: "EDEVICE", -4: "ERANGE", -5: "EUNSUPPORTED"}

EXPORTED = ["blco_build", "blco_mttkrp", "blco_mttkrp_acc", "blco_mttkrp_v", "blco_mttkrp_stream",
            "blco_mttkrp_stream_all", "blco_mttkrp_ws", "blco_mttkrp_stream_all_ws",
            "blco_cp_grad_ws", "blco_workspace", "blco_build_device_in", "blco_build_device_sizes",
            "blco_sampled_loss", "blco_cp_grad", "blco_cp_grad_noalloc", "blco_scale", "blco_cast_bf16", "blco_set_resolution", "blco_resolution",
            "blco_plan", "blco_stream_plan", "blco_scale_all", "blco_cast_bf16_all", "blco_cp_als_in", "blco_cp_als_size",
            "blco_gram", "blco_cp_als", "blco_build_device",
            "blco_atomic_probe", "blco_gather_probe", "blco_frequent_rows", "blco_info", "blco_export", "blco_free",
            "blco_last_error"]


class BLCOError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__(f"{STATUS.get(code, code)}: {msg}")
        self.code = code
        self.status = STATUS.get(code, str(code))


class _Opts(ctypes.Structure):
    _fields_ = [("key_bits", ctypes.c_int), ("max_block_nnz", ctypes.c_int64),
                ("placement", ctypes.c_int), ("hot_min_count", ctypes.c_int64)]


class _CPALSOpts(ctypes.Structure):
    _fields_ = [("max_iters", ctypes.c_int), ("tol", ctypes.c_double), ("factor_dtype", ctypes.c_int)]


class _CPALSReport(ctypes.Structure):
    _fields_ = [("iters", ctypes.c_int), ("pinv_fallbacks", ctypes.c_int)]


class _Info(ctypes.Structure):
    _fields_ = [("nmodes", ctypes.c_int), ("nnz", ctypes.c_int64), ("total_bits", ctypes.c_int),
                ("key_bits", ctypes.c_int), ("block_bits", ctypes.c_int),
                ("bits", ctypes.c_int * MAX_MODES), ("kept", ctypes.c_int * MAX_MODES),
                ("shift", ctypes.c_int * MAX_MODES), ("high", ctypes.c_int * MAX_MODES),
                ("dims", ctypes.c_uint64 * MAX_MODES), ("nblocks", ctypes.c_int64),
                ("nruns", ctypes.c_int64), ("placement", ctypes.c_int),
                ("device_bytes", ctypes.c_size_t), ("host_bytes", ctypes.c_size_t),
                ("stream_peak_bytes", ctypes.c_size_t), ("stream_chunks", ctypes.c_int64),
                ("stream_chunk_nnz", ctypes.c_int64), ("stream_copy_ms", ctypes.c_double),
                ("stream_kernel_ms", ctypes.c_double), ("stream_total_ms", ctypes.c_double),
                ("hot_rows", ctypes.c_int * MAX_MODES),
                ("build_stage_ms", ctypes.c_double * 5)]


class _Plan(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int) for k in
                ("resolution", "lanes", "ranks_per_lane", "window", "wpt", "stash_rows", "copies",
                 "wide", "vector_gathers", "factor_stride", "out_stride", "out_copies", "grouped")] + [
                    ("workgroups", ctypes.c_int64), ("workspace_bytes", ctypes.c_size_t),
                    ("flushes", ctypes.c_double * 2)]


def library_path() -> str:
    return _SO


def lib():
    """The loaded ``libblco.so``; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(_SO):
            raise RuntimeError(f"{_SO} is missing: build it with `python -m paper_2201_12523_amd.buildlib`")
        L = ctypes.CDLL(_SO)
        p, i64, i32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
        L.blco_build.argtypes = [i32, p, i64, p, p, p, ctypes.POINTER(p)]
        L.blco_mttkrp.argtypes = [p, i32, p, i32, i32, p, p]
        L.blco_mttkrp_acc.argtypes = [p, i32, p, i32, i32, p, p]
        L.blco_mttkrp_v.argtypes = [p, i32, p, p, i32, i32, p, ctypes.c_double, p, p]
        L.blco_mttkrp_stream.argtypes = [p, i32, p, i32, i32, p, ctypes.c_size_t, p]
        L.blco_mttkrp_stream_all.argtypes = [p, p, i32, i32, p, ctypes.c_size_t, p]
        sz = ctypes.c_size_t
        L.blco_mttkrp_ws.argtypes = [p, i32, p, p, i32, i32, p, ctypes.c_double, i32, p, p, sz, p]
        L.blco_mttkrp_stream_all_ws.argtypes = [p, p, i32, i32, p, sz, p, sz, p]
        L.blco_cp_grad_ws.argtypes = [p, p, i32, i32, p, ctypes.c_double, p, p, p, sz, p, sz, p]
        L.blco_workspace.argtypes = [p, i32, i32, i32, ctypes.POINTER(sz)]
        L.blco_plan.argtypes = [p, i32, i32, i32, i32, i64, sz, ctypes.POINTER(_Plan)]
        L.blco_stream_plan.argtypes = [p, ctypes.c_uint, i32, i32, i32, sz, sz, ctypes.POINTER(sz),
                                       ctypes.POINTER(i64)]
        L.blco_sampled_loss.argtypes = [p, p, i32, i32, p, p, p]
        L.blco_cast_bf16.argtypes = [p, p, i64, p]
        L.blco_cast_bf16_all.argtypes = [i32, p, p, p, p]
        L.blco_scale_all.argtypes = [i32, p, p, p, ctypes.c_double, p]
        L.blco_cp_grad.argtypes = [p, p, i32, i32, p, ctypes.c_double, p, p, p, ctypes.c_size_t,
                                   p]
        L.blco_cp_grad_noalloc.argtypes = [p, p, i32, i32, p, ctypes.c_double, p, p, p, p]
        L.blco_scale.argtypes = [p, i64, p, ctypes.c_double, p]
        L.blco_info.argtypes = [p, ctypes.POINTER(_Info)]
        L.blco_export.argtypes = [p, p, p, p, p]
        L.blco_set_resolution.argtypes = [p, i32]
        L.blco_build_device.argtypes = [i32, p, i64, p, p, ctypes.POINTER(_Opts), p,
                                        ctypes.POINTER(p)]
        L.blco_build_device_in.argtypes = [i32, p, i64, p, p, ctypes.POINTER(_Opts), p, sz, p, sz, p,
                                           ctypes.POINTER(p)]
        L.blco_build_device_sizes.argtypes = [i32, p, i64, ctypes.POINTER(_Opts),
                                              ctypes.POINTER(sz), ctypes.POINTER(sz)]
        L.blco_gram.argtypes = [p, i32, i64, i32, p, p]
        L.blco_cp_als_in.argtypes = [p, p, i32, p, p, p, p, sz, p]
        L.blco_cp_als_size.argtypes = [p, i32, i32, ctypes.POINTER(sz)]
        L.blco_cp_als.argtypes = [p, p, i32, ctypes.POINTER(_CPALSOpts), p,
                                  ctypes.POINTER(_CPALSReport), p]
        L.blco_resolution.argtypes = [p, i32, i32, ctypes.POINTER(ctypes.c_int)]
        L.blco_frequent_rows.argtypes = [p, i32, i32, ctypes.POINTER(ctypes.c_int)]
        L.blco_atomic_probe.argtypes = [p, i64, i32, p, i64, p]
        L.blco_gather_probe.argtypes = [p, i64, i32, p, i64, p, p]
        L.blco_free.argtypes = [p]
        L.blco_free.restype = None
        L.blco_last_error.restype = ctypes.c_char_p
        for name in EXPORTED:
            if name not in ("blco_free", "blco_last_error"):
                getattr(L, name).restype = ctypes.c_int
        _lib = L
    return _lib


def _check(rc):
    if rc != 0:
        raise BLCOError(rc, lib().blco_last_error().decode())


def _torch_stream(stream):
    """A caller's stream as torch takes it (None stays None): anything with a `cuda_stream` handle
    is a stream to this package."""
    if stream is None or isinstance(stream, torch.cuda.Stream):
        return stream
    return torch.cuda.ExternalStream(int(stream.cuda_stream))


def _stream(stream=None, t=None) -> int:
    """The stream handle of a call.  A tensor whose arrays live in a torch allocation made on
    another stream is recorded on this one, so that its memory is not reused before the
    call's work has run."""
    if stream is None:
        stream = torch.cuda.current_stream()
    h = int(stream.cuda_stream)
    if t is not None and t._storage is not None and h != t._storage_stream:
        t._storage.record_stream(_torch_stream(stream))
    return h


def _with_memory(call):
    """call() again after torch has released its cached blocks, where device memory ran out
    (the library's own allocations do not reach into torch's cache; it makes them before it
    writes anything)."""
    rc = call()
    if rc == -2 and not lib().blco_last_error().startswith(b"budget") and torch.cuda.is_available():
        if not torch.cuda.is_current_stream_capturing():
            torch.cuda.empty_cache()
            rc = call()
    return rc


RESOLUTIONS = {"auto": 0, "register": 1, "hierarchical": 2}


class BLCOTensor:
    """A BLCO tensor owned by the library (freed with the object)."""

    def __init__(self, handle, dims, storage=None, storage_stream=0):
        self._h = ctypes.c_void_p(handle)
        self.dims = tuple(int(d) for d in dims)
        self._storage = storage               # torch memory that holds the tensor's arrays
        self._storage_stream = storage_stream
        self._fixed = None                    # (nnz, placement): they never change
        self._need = {}                       # workspace bytes by (mode, rank, dtype)

    @property
    def handle(self):
        return self._h

    def _facts(self):
        if self._fixed is None or self._h is None:
            inf = self.info()
            self._fixed = inf["nnz"], inf["placement"]
        return self._fixed

    def info(self) -> dict:
        inf = _Info()
        _check(lib().blco_info(self._h, ctypes.byref(inf)))
        N = inf.nmodes
        return dict(nmodes=N, nnz=inf.nnz, total_bits=inf.total_bits, key_bits=inf.key_bits,
                    block_bits=inf.block_bits, bits=list(inf.bits[:N]), kept=list(inf.kept[:N]),
                    shift=list(inf.shift[:N]), high=list(inf.high[:N]), dims=list(inf.dims[:N]),
                    nblocks=inf.nblocks, nruns=inf.nruns, placement=inf.placement,
                    device_bytes=inf.device_bytes, host_bytes=inf.host_bytes,
                    stream_peak_bytes=inf.stream_peak_bytes, stream_chunks=inf.stream_chunks,
                    stream_chunk_nnz=inf.stream_chunk_nnz, stream_copy_ms=inf.stream_copy_ms,
                    stream_kernel_ms=inf.stream_kernel_ms, stream_total_ms=inf.stream_total_ms,
                    hot_rows=list(inf.hot_rows[:N]),
                    build_stage_ms=dict(zip(("linearize", "sort", "encode", "runs",
                                             "frequent_rows"), list(inf.build_stage_ms))))

    @property
    def nnz(self) -> int:
        return self._facts()[0]

    @property
    def nmodes(self) -> int:
        return len(self.dims)

    def set_resolution(self, resolution: str):
        """Conflict resolution of later MTTKRP calls: "auto" (Section 5.3 heuristic),
        "register" (Section 5.2) or "hierarchical" (Section 5.1)."""
        if resolution not in RESOLUTIONS:
            raise ValueError(f"resolution {resolution!r}: one of {sorted(RESOLUTIONS)}")
        _check(lib().blco_set_resolution(self._h, RESOLUTIONS[resolution]))
        self._need = {}

    def resolution(self, mode: int, rank: int) -> str:
        """The mechanism a mode-`mode` MTTKRP at rank `rank` uses on the current device."""
        c = ctypes.c_int(-1)
        _check(lib().blco_resolution(self._h, int(mode), int(rank), ctypes.byref(c)))
        return {v: k for k, v in RESOLUTIONS.items()}[c.value]

    def stash_rows(self, mode: int, rank: int) -> int:
        """Frequent rows of `mode` a register-based MTTKRP at `rank` sums in its LDS stash."""
        c = ctypes.c_int(-1)
        _check(lib().blco_frequent_rows(self._h, int(mode), int(rank), ctypes.byref(c)))
        return c.value

    def workspace(self, mode: int, rank: int, dtype: str = "fp32") -> int:
        """Bytes of workspace a mode-`mode` MTTKRP at `rank` takes (mode -1: a call over every
        mode); the functions of this module allocate it themselves."""
        n = ctypes.c_size_t()
        _check(lib().blco_workspace(self._h, int(mode), int(rank), BF16 if dtype == "bf16" else F32,
                                    ctypes.byref(n)))
        return n.value

    def plan(self, mode: int, rank: int, dtype: str = "fp32", use: str = "mttkrp", nnz: int = 0,
             workspace=None) -> dict:
        """How a launch of `mode` at `rank` runs (blco_plan): window, lanes, frequent rows, padding.
        use: "mttkrp", "residual" (the CP gradient's fused walk) or "als"; nnz: non-zeros of the
        launch (0: the tensor's); workspace: bytes lent (None: as many as it wants)."""
        pl = _Plan()
        _check(lib().blco_plan(self._h, int(mode), int(rank), BF16 if dtype == "bf16" else F32,
                               {"mttkrp": 0, "residual": 1, "als": 2}[use], int(nnz),
                               (1 << 62) if workspace is None else int(workspace),
                               ctypes.byref(pl)))
        out = {k: getattr(pl, k) for k, _ in _Plan._fields_}
        out["flushes"] = tuple(pl.flushes)
        return out

    def export(self):
        """(keys uint64, values float32, block_ids uint64, block_starts int64) on the host."""
        inf = self.info()
        n, nb = inf["nnz"], inf["nblocks"]
        keys = np.empty(n, dtype=np.uint64)
        vals = np.empty(n, dtype=np.float32)
        bids = np.empty(nb, dtype=np.uint64)
        bst = np.empty(nb + 1, dtype=np.int64)
        _check(lib().blco_export(self._h, keys.ctypes.data, vals.ctypes.data, bids.ctypes.data,
                                 bst.ctypes.data))
        return keys, vals, bids, bst

    def free(self):
        if self._h is not None and self._h.value:
            lib().blco_free(self._h)
        self._h = None
        self._storage = None

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


def build(coords, values, dims, key_bits=64, max_block_nnz=1 << 27, placement="device",
          hot_min_count=0):
    """Build a BLCO tensor from 0-based COO coordinates (list of N integer arrays) and values.

    hot_min_count: non-zeros a row needs to count as frequent (0: the library's
    default; negative: no frequent rows)."""
    N = len(dims)
    cs = [np.ascontiguousarray(c, dtype=np.uint32) for c in coords]
    if len(cs) != N:
        raise ValueError("one coordinate array per mode")
    v = np.ascontiguousarray(values, dtype=np.float32)
    d = np.ascontiguousarray(dims, dtype=np.uint64)
    arr = (ctypes.c_void_p * N)(*[c.ctypes.data for c in cs])
    opts = _Opts(key_bits, max_block_nnz, PLACEMENTS[placement], int(hot_min_count))
    h = ctypes.c_void_p()
    _check(_with_memory(lambda: lib().blco_build(N, d.ctypes.data, len(v), arr, v.ctypes.data,
                                                 ctypes.byref(opts), ctypes.byref(h))))
    return BLCOTensor(h.value, dims)


def build_device(coords, values, dims, key_bits=64, max_block_nnz=1 << 27, placement="device",
                 hot_min_count=0, stream=None):
    """blco_build on the GPU.  coords: N index arrays (numpy, or int32 device tensors holding
    the uint32 bits); values: float32 (numpy or device tensor).  Same result as build()."""
    N = len(dims)
    if len(coords) != N:
        raise ValueError("one coordinate array per mode")
    dev = torch.device("cuda", torch.cuda.current_device())
    keep = []
    for c in coords:
        if isinstance(c, torch.Tensor):
            if not c.is_cuda or c.dtype != torch.int32 or not c.is_contiguous():
                raise ValueError("device coordinates must be contiguous int32 tensors")
            keep.append(c)
        else:
            a = np.ascontiguousarray(c, dtype=np.uint32).view(np.int32)
            keep.append(torch.from_numpy(a).to(dev))
    if isinstance(values, torch.Tensor):
        if not values.is_cuda or values.dtype != torch.float32 or not values.is_contiguous():
            raise ValueError("device values must be a contiguous float32 tensor")
        v = values
    else:
        v = torch.from_numpy(np.ascontiguousarray(values, dtype=np.float32)).to(dev)
    nnz = v.numel()
    for c in keep:
        if c.numel() != nnz:
            raise ValueError("coordinate arrays and values differ in length")
    d = np.ascontiguousarray(dims, dtype=np.uint64)
    arr = (ctypes.c_void_p * N)(*[c.data_ptr() for c in keep])
    opts = _Opts(key_bits, max_block_nnz, PLACEMENTS[placement], int(hot_min_count))
    h = ctypes.c_void_p()
    need_s, need_w = ctypes.c_size_t(), ctypes.c_size_t()
    _check(lib().blco_build_device_sizes(N, d.ctypes.data, nnz, ctypes.byref(opts),
                                         ctypes.byref(need_s), ctypes.byref(need_w)))
    # the arrays and the workspace from the pool of the stream the build runs on
    sh = _stream(stream)
    storage = ws = None
    with torch.cuda.stream(_torch_stream(stream)):
        try:
            if need_s.value:
                storage = torch.empty(need_s.value, dtype=torch.uint8, device=dev)
            ws = torch.empty(need_w.value, dtype=torch.uint8, device=dev)
        except torch.cuda.OutOfMemoryError:
            pass   # the library allocates what it was not given, or says what it could not
    blk = lambda x: (None, 0) if x is None else (x.data_ptr(), x.numel())
    _check(_with_memory(lambda: lib().blco_build_device_in(
        N, d.ctypes.data, nnz, arr, v.data_ptr(), ctypes.byref(opts), *blk(storage), *blk(ws), sh,
        ctypes.byref(h))))
    return BLCOTensor(h.value, dims, storage, sh)


_DTYPES = {torch.float32: F32, torch.bfloat16: BF16}


def _factor_args(t, factors, mode_skip):
    dt = None
    R = None
    ptrs = []
    keep = []
    dims = t.dims
    for m, f in enumerate(factors):
        if f is None:
            ptrs.append(None)
            continue
        shape = f.shape
        if not f.is_cuda or not f.is_contiguous() or len(shape) != 2:
            raise ValueError(f"factor {m} must be a contiguous 2-D device tensor")
        if shape[0] != dims[m]:
            raise ValueError(f"factor {m} has {shape[0]} rows, mode length is {dims[m]}")
        fd = _DTYPES.get(f.dtype)
        if fd is None:
            raise ValueError("factors must be float32 or bfloat16")
        if dt is None:
            dt, R = fd, int(shape[1])
        elif fd != dt or shape[1] != R:
            raise ValueError("all factors must share dtype and rank")
        ptrs.append(f.data_ptr())
        keep.append(f)
    if R is None:
        raise ValueError("no factor given")
    return (ctypes.c_void_p * len(factors))(*ptrs), dt, R, keep


def _out(t, mode, R, out, device):
    if out is None:
        out = torch.empty((t.dims[mode], R), dtype=torch.float32, device=device)
    elif (out.dtype != torch.float32 or not out.is_contiguous() or
          tuple(out.shape) != (t.dims[mode], R)):
        raise ValueError("out must be a contiguous float32 tensor of shape (I_mode, R)")
    return out


def _workspace(t, mode, R, dt, device, stream):
    """(tensor or None, pointer, bytes): the workspace a call of `mode` (-1: all) can use, from
    torch's allocator in the stream's order; none where memory is short."""
    bytes_ = t._need.get((mode, R, dt)) if t._h is not None else None
    if bytes_ is None:
        need = ctypes.c_size_t()
        _check(lib().blco_workspace(t.handle, mode, R, dt, ctypes.byref(need)))
        bytes_ = t._need[(mode, R, dt)] = need.value
    return _lend(bytes_, device, stream)


def _stream_workspace(t, modes, gradient, R, dt, budget, device, stream):
    """The workspace a call under a device budget uses; none where the budget has no room, and
    where the call itself will say what is wrong with its arguments."""
    used, chunk = ctypes.c_size_t(), ctypes.c_int64()
    bits = sum(1 << m for m in set(modes) if 0 <= m < len(t.dims))
    if lib().blco_stream_plan(t.handle, bits, gradient, R, dt, int(budget), 1 << 62,
                              ctypes.byref(used), ctypes.byref(chunk)) != 0:
        return None, None, 0
    return _lend(used.value, device, stream)


def _lend(bytes_, device, stream):
    """(tensor or None, pointer, bytes) of a block from the pool of the stream a call runs on."""
    if bytes_ == 0:
        return None, None, 0
    try:
        # from the pool of the stream the call runs on: blocks there are reused in its order
        if stream is None:
            ws = torch.empty(bytes_, dtype=torch.uint8, device=device)
        else:
            with torch.cuda.stream(_torch_stream(stream)):
                ws = torch.empty(bytes_, dtype=torch.uint8, device=device)
    except torch.cuda.OutOfMemoryError:
        return None, None, 0
    return ws, ws.data_ptr(), bytes_


def _device_of(factors):
    for f in factors:
        if f is not None:
            return f.device
    return torch.device("cuda")


def mttkrp(t, mode, factors, out=None, stream=None):
    """Mode-``mode`` MTTKRP of an in-memory BLCO tensor; returns out (I_mode x R, float32)."""
    arr, dt, R, _keep = _factor_args(t, factors, mode)
    out = _out(t, mode, R, out, _device_of(factors))
    ws, wp, wb = _workspace(t, mode, R, dt, out.device, stream)
    _check(lib().blco_mttkrp_ws(t.handle, mode, None, arr, dt, R, None, 1.0, 0, out.data_ptr(), wp,
                                wb, _stream(stream, t)))
    return out


def mttkrp_acc(t, mode, factors, out, stream=None):
    """out += mode-``mode`` MTTKRP (out is not cleared first)."""
    arr, dt, R, _keep = _factor_args(t, factors, mode)
    out = _out(t, mode, R, out, _device_of(factors))
    ws, wp, wb = _workspace(t, mode, R, dt, out.device, stream)
    _check(lib().blco_mttkrp_ws(t.handle, mode, None, arr, dt, R, None, 1.0, 1, out.data_ptr(), wp,
                                wb, _stream(stream, t)))
    return out


def mttkrp_v(t, mode, values, factors, out=None, scale=None, alpha=1.0, stream=None):
    """MTTKRP with the values replaced (device float32, BLCO order), scaled by alpha*scale."""
    arr, dt, R, _keep = _factor_args(t, factors, mode)
    out = _out(t, mode, R, out, _device_of(factors))
    if values.dtype != torch.float32 or not values.is_contiguous():
        raise ValueError("values must be contiguous float32")
    sp = None
    if scale is not None:
        if scale.dtype != torch.float64 or scale.numel() != 1:
            raise ValueError("scale must be a one-element float64 device tensor")
        sp = scale.data_ptr()
    ws, wp, wb = _workspace(t, mode, R, dt, out.device, stream)
    _check(lib().blco_mttkrp_ws(t.handle, mode, values.data_ptr(), arr, dt, R, sp, float(alpha), 0,
                                out.data_ptr(), wp, wb, _stream(stream, t)))
    return out


def mttkrp_stream(t, mode, factors, out=None, device_budget=8_000_000_000, stream=None):
    """MTTKRP of a tensor in pinned host memory, streamed under a device-memory budget."""
    arr, dt, R, _keep = _factor_args(t, factors, mode)
    out = _out(t, mode, R, out, _device_of(factors))
    ws, wp, wb = _stream_workspace(t, [mode], 0, R, dt, device_budget, out.device, stream)
    if wb == 0:
        _check(_with_memory(lambda: lib().blco_mttkrp_stream(
            t.handle, mode, arr, dt, R, out.data_ptr(), int(device_budget), _stream(stream, t))))
        return out
    outs = (ctypes.c_void_p * len(t.dims))()
    outs[mode] = out.data_ptr()
    _check(_with_memory(lambda: lib().blco_mttkrp_stream_all_ws(
        t.handle, arr, dt, R, outs, int(device_budget), wp, wb, _stream(stream, t))))
    return out


def mttkrp_stream_all(t, factors, outs=None, device_budget=8_000_000_000, modes=None,
                      stream=None):
    """MTTKRP of several modes (default: all) in one streamed pass over a pinned tensor."""
    arr, dt, R, _keep = _factor_args(t, factors, None)
    dev = _device_of(factors)
    modes = list(range(len(t.dims))) if modes is None else list(modes)
    if outs is None:
        outs = [None] * len(t.dims)
    outs = list(outs)
    for m in modes:
        outs[m] = _out(t, m, R, outs[m], dev)
    ptrs = (ctypes.c_void_p * len(t.dims))(*[outs[m].data_ptr() if m in modes else None
                                               for m in range(len(t.dims))])
    ws, wp, wb = _stream_workspace(t, modes, 0, R, dt, device_budget, dev, stream)
    _check(_with_memory(lambda: lib().blco_mttkrp_stream_all_ws(
        t.handle, arr, dt, R, ptrs, int(device_budget), wp, wb, _stream(stream, t))))
    return [outs[m] if m in modes else None for m in range(len(t.dims))]


def sampled_loss(t, factors, residual=None, loss=None, stream=None):
    """(loss, residual): 1/2 sum_k (x_k - xhat_k)^2 as a float64 device scalar, and e (BLCO order)."""
    arr, dt, R, _keep = _factor_args(t, factors, None)
    dev = _device_of(factors)
    n = t.nnz
    if residual is None:
        residual = torch.empty(n, dtype=torch.float32, device=dev)
    if loss is None:
        loss = torch.empty((), dtype=torch.float64, device=dev)
    _check(_with_memory(lambda: lib().blco_sampled_loss(
        t.handle, arr, dt, R, residual.data_ptr(), loss.data_ptr(), _stream(stream, t))))
    return loss, residual


def cp_grad(t, factors, grads=None, residual=None, loss=None, scale=None, alpha=1.0,
            device_budget=8_000_000_000, stream=None):
    """(loss, grads, residual): the sparse CP fit loss 1/2 sum_k e_k^2 (float64 device scalar)
    and alpha * scale * dloss/dA^(m) = -alpha * scale * MTTKRP_m(E) for every mode, in one call.

    A device tensor also returns the residual e (BLCO order); a tensor in pinned host
    memory is streamed under `device_budget` (residual None)."""
    arr, dt, R, _keep = _factor_args(t, factors, None)
    dev = _device_of(factors)
    N = len(t.dims)
    if grads is None:
        grads = [None] * N
    grads = [_out(t, m, R, grads[m], dev) for m in range(N)]
    pinned = t._facts()[1] == PLACEMENTS["pinned"]
    if not pinned and residual is None:
        residual = torch.empty(max(t.nnz, 1), dtype=torch.float32, device=dev)
    if loss is None:
        loss = torch.empty((), dtype=torch.float64, device=dev)
    sp = None
    if scale is not None:
        if scale.dtype != torch.float64 or scale.numel() != 1:
            raise ValueError("scale must be a one-element float64 device tensor")
        sp = scale.data_ptr()
    ptrs = (ctypes.c_void_p * N)(*[g.data_ptr() for g in grads])
    if pinned:
        ws, wp, wb = _stream_workspace(t, range(N), 1, R, dt, device_budget, dev, stream)
    else:
        ws, wp, wb = _workspace(t, -1, R, dt, dev, stream)
    _check(_with_memory(lambda: lib().blco_cp_grad_ws(
        t.handle, arr, dt, R, sp, float(alpha), None if pinned else residual.data_ptr(),
        loss.data_ptr(), ptrs, int(device_budget), wp, wb, _stream(stream, t))))
    return loss, grads, (None if pinned else residual)


def cp_grad_noalloc(t, factors, grads, residual, loss, scale=None, alpha=1.0, stream=None):
    """cp_grad for a device tensor through the entry point that allocates nothing on the
    device: every output (grads, residual of t.nnz floats, a float64 loss) is the caller's."""
    arr, dt, R, _keep = _factor_args(t, factors, None)
    N = len(t.dims)
    if len(grads) != N:
        raise ValueError(f"{N} gradients expected")
    sp = None
    if scale is not None:
        if scale.dtype != torch.float64 or scale.numel() != 1:
            raise ValueError("scale must be a one-element float64 device tensor")
        sp = scale.data_ptr()
    ptrs = (ctypes.c_void_p * N)(*[g.data_ptr() for g in grads])
    _check(lib().blco_cp_grad_noalloc(t.handle, arr, dt, R, sp, float(alpha), residual.data_ptr(),
                                      loss.data_ptr(), ptrs, _stream(stream, t)))
    return loss, grads, residual


def scale_(x, scale, alpha=1.0, stream=None):
    """x *= alpha * scale (x float32 device tensor, scale a one-element float64 device tensor)."""
    if x.dtype != torch.float32 or not x.is_contiguous():
        raise ValueError("x must be contiguous float32")
    if scale.dtype != torch.float64 or scale.numel() != 1:
        raise ValueError("scale must be a one-element float64 device tensor")
    _check(lib().blco_scale(x.data_ptr(), x.numel(), scale.data_ptr(), float(alpha),
                            _stream(stream)))
    return x


def _arrays(xs):
    """Pointers and lengths of tensors, as the calls over several arrays take them."""
    return ((ctypes.c_void_p * len(xs))(*[x.data_ptr() for x in xs]),
            (ctypes.c_int64 * len(xs))(*[x.numel() for x in xs]))


def _scale_all(xs, scale):
    """scale_ of every tensor of a list, in one launch."""
    ptrs, n = _arrays(xs)
    _check(lib().blco_scale_all(len(xs), ptrs, n, scale.data_ptr(), 1.0, _stream()))


def _cast_all(xs):
    """cast_bf16 of every tensor of a list, in one launch."""
    for x in xs:
        if x.dtype != torch.float32:
            raise ValueError("x must be contiguous float32")
    ys = [torch.empty(x.shape, dtype=torch.bfloat16, device=x.device) for x in xs]
    src, n = _arrays(xs)
    _check(lib().blco_cast_bf16_all(len(xs), src, _arrays(ys)[0], n, _stream()))
    return ys


def cast_bf16(x, stream=None):
    """Round-to-nearest-even bfloat16 copy of a float32 device tensor (library kernel)."""
    if x.dtype != torch.float32 or not x.is_contiguous():
        raise ValueError("x must be contiguous float32")
    y = torch.empty(x.shape, dtype=torch.bfloat16, device=x.device)
    _check(lib().blco_cast_bf16(x.data_ptr(), y.data_ptr(), x.numel(), _stream(stream)))
    return y


def atomic_probe(out, rows, stream=None):
    """Calibration kernel: out[rows[k], :] += 1 with one device-scope fp32 atomic per entry
    (16-lane groups, the MTTKRP kernels' flush pattern).  out: float32 (I x R) device
    tensor; rows: int32 device tensor of row ids (uint32 bits)."""
    if out.dtype != torch.float32 or not out.is_contiguous() or out.dim() != 2:
        raise ValueError("out must be a contiguous 2-D float32 tensor")
    if rows.dtype != torch.int32 or not rows.is_contiguous():
        raise ValueError("rows must be a contiguous int32 tensor")
    _check(lib().blco_atomic_probe(out.data_ptr(), out.shape[0], out.shape[1], rows.data_ptr(),
                                   rows.numel(), _stream(stream)))
    return out


def gather_probe(table, rows, sink, stream=None):
    """Calibration kernel: reads table[rows[k], :] by 16-lane groups, six rows per group in
    flight (the MTTKRP kernels' gather pattern), one partial sum per group into sink.
    table: float32 (I x R) device tensor; rows: int32 device tensor of row ids (uint32
    bits); sink: float32 device tensor of at least ceil(len(rows) / 6) entries."""
    if table.dtype != torch.float32 or not table.is_contiguous() or table.dim() != 2:
        raise ValueError("table must be a contiguous 2-D float32 tensor")
    if rows.dtype != torch.int32 or not rows.is_contiguous():
        raise ValueError("rows must be a contiguous int32 tensor")
    if sink.dtype != torch.float32 or sink.numel() < (rows.numel() + 5) // 6:
        raise ValueError("sink must be a float32 tensor of at least ceil(len(rows) / 6) entries")
    _check(lib().blco_gather_probe(table.data_ptr(), table.shape[0], table.shape[1],
                                   rows.data_ptr(), rows.numel(), sink.data_ptr(),
                                   _stream(stream)))
    return sink


def gram(A, stream=None):
    """A^T A as a float64 R x R device tensor (fp32 products, fp64 sums; library kernel)."""
    if A.dim() != 2 or not A.is_contiguous() or A.dtype not in (torch.float32, torch.bfloat16):
        raise ValueError("A must be a contiguous 2-D float32 or bfloat16 tensor")
    R = A.shape[1]
    G = torch.empty((R, R), dtype=torch.float64, device=A.device)
    dt = BF16 if A.dtype == torch.bfloat16 else F32
    _check(lib().blco_gram(A.data_ptr(), dt, A.shape[0], R, G.data_ptr(), _stream(stream)))
    return G


def cp_als(t, factors, max_iters=25, tol=1e-5, storage="fp32", stream=None):
    """CP-ALS (Algorithm 1) on the device; `factors` (fp32 I_m x R device tensors) are the
    initial values and are overwritten.  Returns (fits per iteration, report dict)."""
    for f in factors:
        if f.dtype != torch.float32 or not f.is_contiguous() or f.dim() != 2:
            raise ValueError("factors must be contiguous 2-D float32 tensors")
    R = factors[0].shape[1]
    arr = (ctypes.c_void_p * len(factors))(*[f.data_ptr() for f in factors])
    if storage not in ("fp32", "bf16"):
        raise ValueError("storage must be 'fp32' or 'bf16'")
    for m, f in enumerate(factors):
        if f.shape[0] != t.dims[m] or f.shape[1] != R:
            raise ValueError(f"factor {m} must be {t.dims[m]} x {R}")
    opts = _CPALSOpts(int(max_iters), float(tol), BF16 if storage == "bf16" else F32)
    fits = np.zeros(int(max_iters), dtype=np.float64)
    rep = _CPALSReport()
    sh = _stream(stream, t)
    need, ws = ctypes.c_size_t(), None
    if lib().blco_cp_als_size(t.handle, R, opts.factor_dtype, ctypes.byref(need)) == 0:
        # from the pool of the stream the call runs on; the call itself says what is wrong
        # with its arguments, and allocates where this cannot
        try:
            with torch.cuda.stream(_torch_stream(stream)):
                ws = torch.empty(need.value, dtype=torch.uint8, device=factors[0].device)
        except torch.cuda.OutOfMemoryError:
            pass
    wp, wb = (None, 0) if ws is None else (ws.data_ptr(), need.value)
    _check(_with_memory(lambda: lib().blco_cp_als_in(t.handle, arr, R, ctypes.byref(opts),
                                                     fits.ctypes.data, ctypes.byref(rep), wp, wb,
                                                     sh)))
    return fits[:rep.iters].tolist(), {"iters": rep.iters, "pinv_fallbacks": rep.pinv_fallbacks}


class CPLoss(torch.autograd.Function):
    """Sparse CP fit loss 1/2 sum_nnz (x - sum_r prod_m A^(m))^2 with a hand-written backward.

    forward(t, storage, *A): A are fp32 factor masters (I_m x R); storage "fp32"
    or "bf16" (round-to-nearest-even copies used by the kernels).  The loss is a
    float64 device scalar.  When any factor needs a gradient, the forward makes one
    blco_cp_grad call: the loss and dL/dA^(m) = -MTTKRP_m(E) for every mode (E the
    residual tensor), the residual formed inside one mode's MTTKRP walk; the backward
    then only scales them by the incoming gradient g.  Otherwise the forward runs the
    sampled-loss kernel alone.  A tensor in pinned host memory is streamed (budget:
    CPLoss.device_budget bytes).
    """

    device_budget = 8_000_000_000

    @staticmethod
    def forward(ctx, t, storage, *A):
        if storage == "bf16":
            F = _cast_all([a.contiguous() for a in A])
        elif storage == "fp32":
            F = [a.contiguous() for a in A]
        else:
            raise ValueError("storage must be 'fp32' or 'bf16'")
        pinned = t._facts()[1] == PLACEMENTS["pinned"]
        if any(ctx.needs_input_grad[2:]) or pinned:
            loss, grads, _ = cp_grad(t, F, device_budget=CPLoss.device_budget)
            ctx.grads = grads
        else:
            loss, _ = sampled_loss(t, F)
            ctx.grads = None
        return loss

    @staticmethod
    def backward(ctx, g):
        g = g.detach().reshape(1)
        if g.dtype != torch.float64:
            raise ValueError("loss gradient must be float64")
        g = g.contiguous()
        grads = ctx.grads
        ctx.grads = None
        _scale_all(grads, g)
        return (None, None, *grads)

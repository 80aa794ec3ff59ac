"""alpha-entmax flash attention for MI355X (gfx950): Python binding.

Argument marshalling over the C ABI declared in include/entmax_attn.h; every
step of the computation runs in the HIP kernels of libentmax_attn.so.  torch
is used only to own device memory and to name the stream.  There is no CPU
fallback: importing this module without the built library raises.

    import paper_2502_12082_amd as ea
    o, res = ea.forward(q, k, v, alpha=1.5, scale=d ** -0.5, causal=False)
    dq, dk, dv = ea.backward(q, k, v, do, res)
"""
from __future__ import annotations

import ctypes
import os
import threading

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libentmax_attn.so")

if not os.path.exists(LIB_PATH):
    raise ImportError("libentmax_attn.so is not built; run `python paper_2502_12082_amd/build.py` "
                      "(or __graft_entry__.build()) first")

# torch ships its own HIP and HSA runtimes.  Importing it first lets the
# library's libamdhip64.so.7 dependency resolve to the copy torch already
# loaded; loaded the other way round the process holds two runtimes, and
# launches through the second one find no device.
import torch  # noqa: E402,F401

_lib = ctypes.CDLL(LIB_PATH)

EA_OK, EA_ERR_INVALID_ARG, EA_ERR_UNSUPPORTED, EA_ERR_WORKSPACE, EA_ERR_HIP = range(5)
EA_BF16, EA_F32 = 0, 1
SYMBOLS = ("entmax_attn_default_params", "entmax_attn_sizes", "entmax_attn_fwd",
           "entmax_attn_bwd", "entmax_attn_fwd_stage", "entmax_attn_bwd_stage",
           "entmax_attn_status_string", "entmax_attn_last_hip_error", "entmax_rows_fwd",
           "entmax_rows_bwd", "entmax_attn_fwd_dense", "entmax_attn_bwd_dense",
           "entmax_attn_bwd_noalloc", "entmax_attn_lists_bytes", "entmax_attn_fwd_lists",
           "entmax_attn_bwd_lists", "entmax_attn_fwd_dense_lists", "entmax_attn_bwd_dense_lists",
           "entmax_attn_bwd_lists_workspace")
EA_ALL_STAGES = -1
NOALLOC_MAX_ROWS = 1048576  # EA_NOALLOC_MAX_ROWS of include/entmax_attn.h


class Shape(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32), ("heads", ctypes.c_int32),
                ("seqlen", ctypes.c_int32), ("head_dim", ctypes.c_int32),
                ("dtype", ctypes.c_int32)]


class Params(ctypes.Structure):
    _fields_ = [("alpha", ctypes.c_float), ("scale", ctypes.c_float),
                ("causal", ctypes.c_int32), ("max_iter", ctypes.c_int32),
                ("tol", ctypes.c_float), ("need_bwd", ctypes.c_int32)]


class ResidualPtrs(ctypes.Structure):
    """The ABI's ea_residuals.  `lists` and `lists_bytes`, set by
    Residuals.ptrs(), name the element lists that belong to them, and `owner`
    the Residuals itself; the calls below then pass those on."""
    lists, lists_bytes, lists_shape, owner = None, 0, None, None
    _fields_ = [(f, ctypes.c_void_p) for f in
                ("tau", "o2", "block_mask", "q_count", "q_index", "k_count", "k_index", "stats",
                 "tau_lo")]


class Sizes(ctypes.Structure):
    _fields_ = [(f, ctypes.c_size_t) for f in
                ("tau", "o2", "block_mask", "q_count", "q_index", "k_count", "k_index", "stats",
                 "ws_fwd", "ws_bwd", "tau_lo")]


_P = ctypes.POINTER
_v = ctypes.c_void_p
_lib.entmax_attn_default_params.argtypes = [_P(Params)]
_lib.entmax_attn_default_params.restype = None
_lib.entmax_attn_sizes.argtypes = [_P(Shape), _P(Params), _P(Sizes)]
_lib.entmax_attn_sizes.restype = ctypes.c_int
_lib.entmax_attn_fwd.argtypes = [_P(Shape), _P(Params), _v, _v, _v, _v, _P(ResidualPtrs), _v,
                                 ctypes.c_size_t, _v]
_lib.entmax_attn_fwd.restype = ctypes.c_int
_lib.entmax_attn_bwd.argtypes = [_P(Shape), _P(Params), _v, _v, _v, _v, _P(ResidualPtrs), _v, _v,
                                 _v, _v, ctypes.c_size_t, _v]
_lib.entmax_attn_bwd.restype = ctypes.c_int
_lib.entmax_attn_fwd_stage.argtypes = [ctypes.c_int, _P(Shape), _P(Params), _v, _v, _v, _v,
                                       _P(ResidualPtrs), _v, ctypes.c_size_t, _v]
_lib.entmax_attn_fwd_stage.restype = ctypes.c_int
_lib.entmax_attn_bwd_stage.argtypes = [ctypes.c_int, _P(Shape), _P(Params), _v, _v, _v, _v,
                                       _P(ResidualPtrs), _v, _v, _v, _v, ctypes.c_size_t, _v]
_lib.entmax_attn_bwd_stage.restype = ctypes.c_int
_lib.entmax_attn_status_string.argtypes = [ctypes.c_int]
_lib.entmax_attn_status_string.restype = ctypes.c_char_p
_lib.entmax_attn_fwd_dense.argtypes = [_P(Shape), _P(Params), _v, _v, _v, _v, _v, _v, _v, _v,
                                       ctypes.c_size_t, _v]
_lib.entmax_attn_fwd_dense.restype = ctypes.c_int
_lib.entmax_attn_bwd_dense.argtypes = [_P(Shape), _P(Params), _v, _v, _v, _v, _v, _v, _v, _v, _v,
                                       _v, _v, ctypes.c_size_t, _v]
_lib.entmax_attn_bwd_dense.restype = ctypes.c_int
_lib.entmax_rows_fwd.argtypes = [ctypes.c_int64, ctypes.c_int32, ctypes.c_int, _P(Params), _v, _v,
                                 _v, _v]
_lib.entmax_rows_fwd.restype = ctypes.c_int
_lib.entmax_rows_bwd.argtypes = [ctypes.c_int64, ctypes.c_int32, ctypes.c_int, _P(Params), _v, _v,
                                 _v, _v, _v]
_lib.entmax_rows_bwd.restype = ctypes.c_int
_lib.entmax_attn_bwd_noalloc.argtypes = [_P(Shape), _P(Params), _v, _v, _v, _v, _P(ResidualPtrs),
                                         _v, _v, _v, _v]
_lib.entmax_attn_bwd_noalloc.restype = ctypes.c_int
_lib.entmax_attn_fwd_dense_lists.argtypes = [_P(Shape), _P(Params), _v, _v, _v, _v, _v, _v, _v, _v,
                                             ctypes.c_size_t, _v, ctypes.c_size_t, _v]
_lib.entmax_attn_fwd_dense_lists.restype = ctypes.c_int
_lib.entmax_attn_bwd_dense_lists.argtypes = [_P(Shape), _P(Params), _v, _v, _v, _v, _v, _v, _v, _v,
                                             ctypes.c_size_t, _v, _v, _v, _v, ctypes.c_size_t, _v]
_lib.entmax_attn_bwd_dense_lists.restype = ctypes.c_int
_lib.entmax_attn_lists_bytes.argtypes = [_P(Shape), _P(Params), _P(ctypes.c_size_t)]
_lib.entmax_attn_lists_bytes.restype = ctypes.c_int
_lib.entmax_attn_bwd_lists_workspace.argtypes = [_P(Shape), _P(Params), _P(ctypes.c_size_t)]
_lib.entmax_attn_bwd_lists_workspace.restype = ctypes.c_int
_lib.entmax_attn_fwd_lists.argtypes = [ctypes.c_int, _P(Shape), _P(Params), _v, _v, _v, _v,
                                       _P(ResidualPtrs), _v, ctypes.c_size_t, _v, ctypes.c_size_t,
                                       _v]
_lib.entmax_attn_fwd_lists.restype = ctypes.c_int
_lib.entmax_attn_bwd_lists.argtypes = [ctypes.c_int, _P(Shape), _P(Params), _v, _v, _v, _v,
                                       _P(ResidualPtrs), _v, ctypes.c_size_t, _v, _v, _v, _v,
                                       ctypes.c_size_t, _v]
_lib.entmax_attn_bwd_lists.restype = ctypes.c_int
_lib.entmax_attn_last_hip_error.argtypes = []
_lib.entmax_attn_last_hip_error.restype = ctypes.c_char_p


class EntmaxAttnError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        msg = "%s: %s (status %d)" % (
            where, _lib.entmax_attn_status_string(status).decode(), status)
        if status == EA_ERR_HIP:
            msg += ": " + _lib.entmax_attn_last_hip_error().decode()
        super().__init__(msg)


def _check(status: int, where: str):
    if status != EA_OK:
        raise EntmaxAttnError(status, where)


# --------------------------------------------------------- raw C ABI calls

def default_params() -> Params:
    p = Params()
    _lib.entmax_attn_default_params(ctypes.byref(p))
    return p


def entmax_attn_sizes(shape: Shape, params: Params) -> Sizes:
    z = Sizes()
    _check(_lib.entmax_attn_sizes(ctypes.byref(shape), ctypes.byref(params), ctypes.byref(z)),
           "entmax_attn_sizes")
    return z


def entmax_attn_lists_bytes(shape: Shape, params: Params) -> int:
    n = ctypes.c_size_t()
    _check(_lib.entmax_attn_lists_bytes(ctypes.byref(shape), ctypes.byref(params), ctypes.byref(n)),
           "entmax_attn_lists_bytes")
    return n.value


def entmax_attn_bwd_lists_workspace(shape: Shape, params: Params) -> int:
    n = ctypes.c_size_t()
    _check(_lib.entmax_attn_bwd_lists_workspace(ctypes.byref(shape), ctypes.byref(params), ctypes.byref(n)),
           "entmax_attn_bwd_lists_workspace")
    return n.value


def _dims(shape):
    return shape.batch, shape.heads, shape.seqlen, shape.head_dim


def _lists_of(res: ResidualPtrs, shape, params):
    """The lists of res, as (pointer, bytes), if they serve this shape."""
    if res.lists is None:
        return None, 0
    if res.lists_shape == _dims(shape):
        return res.lists, res.lists_bytes
    n = ctypes.c_size_t()
    st = _lib.entmax_attn_lists_bytes(ctypes.byref(shape), ctypes.byref(params), ctypes.byref(n))
    return (res.lists, res.lists_bytes) if st == EA_OK and 0 < n.value <= res.lists_bytes else (None, 0)


def entmax_attn_fwd_lists(stage, shape, params, q, k, v, o, res: ResidualPtrs, lists, lists_bytes,
                          workspace, ws_bytes, stream):
    """Raw call; pointers are ints (device addresses), stream an int handle."""
    return _lib.entmax_attn_fwd_lists(stage, ctypes.byref(shape), ctypes.byref(params), q, k, v, o,
                                      ctypes.byref(res), lists, lists_bytes, workspace, ws_bytes,
                                      stream)


def entmax_attn_bwd_lists(stage, shape, params, q, k, v, dout, res: ResidualPtrs, lists,
                          lists_bytes, dq, dk, dv, workspace, ws_bytes, stream):
    return _lib.entmax_attn_bwd_lists(stage, ctypes.byref(shape), ctypes.byref(params), q, k, v,
                                      dout, ctypes.byref(res), lists, lists_bytes, dq, dk, dv,
                                      workspace, ws_bytes, stream)


def entmax_attn_fwd(shape, params, q, k, v, o, res: ResidualPtrs, workspace, ws_bytes, stream):
    lists = _lists_of(res, shape, params)
    if lists[0]:
        return entmax_attn_fwd_lists(EA_ALL_STAGES, shape, params, q, k, v, o, res, *lists, workspace,
                                     ws_bytes, stream)
    return _lib.entmax_attn_fwd(ctypes.byref(shape), ctypes.byref(params), q, k, v, o,
                                ctypes.byref(res), workspace, ws_bytes, stream)


def entmax_attn_bwd(shape, params, q, k, v, dout, res: ResidualPtrs, dq, dk, dv, workspace,
                    ws_bytes, stream):
    lists = _lists_of(res, shape, params)
    if lists[0] and workspace:
        return entmax_attn_bwd_lists(EA_ALL_STAGES, shape, params, q, k, v, dout, res, *lists, dq, dk,
                                     dv, workspace, ws_bytes, stream)
    return _lib.entmax_attn_bwd(ctypes.byref(shape), ctypes.byref(params), q, k, v, dout,
                                ctypes.byref(res), dq, dk, dv, workspace, ws_bytes, stream)


def entmax_attn_bwd_noalloc(shape, params, q, k, v, dout, res: ResidualPtrs, dq, dk, dv, stream):
    """As the C function.  The lists of a Residuals are sorted in a buffer that
    it holds (Residuals.keep_workspace; the first call makes it unless the
    stream is being captured, and without it the lists are not used)."""
    lists = _lists_of(res, shape, params)
    rows = shape.batch * shape.heads * shape.seqlen
    if lists[0] and res.owner is not None and rows <= NOALLOC_MAX_ROWS:
        ws = res.owner.keep_workspace(make=not torch.cuda.is_current_stream_capturing())
        if ws is not None and ws.numel() >= entmax_attn_bwd_lists_workspace(shape, params):
            return entmax_attn_bwd_lists(EA_ALL_STAGES, shape, params, q, k, v, dout, res, *lists, dq,
                                         dk, dv, ws.data_ptr(), ws.numel(), stream)
    return _lib.entmax_attn_bwd_noalloc(ctypes.byref(shape), ctypes.byref(params), q, k, v, dout,
                                        ctypes.byref(res), dq, dk, dv, stream)


def entmax_attn_fwd_stage(stage, shape, params, q, k, v, o, res: ResidualPtrs, workspace,
                          ws_bytes, stream):
    lists = _lists_of(res, shape, params)
    if lists[0] and stage >= 0:
        return entmax_attn_fwd_lists(stage, shape, params, q, k, v, o, res, *lists, workspace,
                                     ws_bytes, stream)
    return _lib.entmax_attn_fwd_stage(stage, ctypes.byref(shape), ctypes.byref(params), q, k, v,
                                      o, ctypes.byref(res), workspace, ws_bytes, stream)


def entmax_attn_bwd_stage(stage, shape, params, q, k, v, dout, res: ResidualPtrs, dq, dk, dv,
                          workspace, ws_bytes, stream):
    lists = _lists_of(res, shape, params)
    if lists[0] and stage >= 0:
        return entmax_attn_bwd_lists(stage, shape, params, q, k, v, dout, res, *lists, dq, dk, dv,
                                     workspace, ws_bytes, stream)
    return _lib.entmax_attn_bwd_stage(stage, ctypes.byref(shape), ctypes.byref(params), q, k, v,
                                      dout, ctypes.byref(res), dq, dk, dv, workspace, ws_bytes,
                                      stream)


# ------------------------------------------------------ torch conveniences

def make_shape(q) -> Shape:
    if q.dim() != 4:
        raise ValueError("expected [batch, heads, seqlen, head_dim]")
    if q.dtype == torch.bfloat16:
        dt = EA_BF16
    elif q.dtype == torch.float32:
        dt = EA_F32
    else:
        raise ValueError("dtype must be bfloat16 or float32")
    B, H, n, d = q.shape
    return Shape(B, H, n, d, dt)


def make_params(alpha=1.5, scale=None, causal=False, need_bwd=True, max_iter=None, tol=None,
                head_dim=64) -> Params:
    p = default_params()
    p.alpha = float(alpha)
    p.scale = float(scale if scale is not None else head_dim ** -0.5)
    p.causal = int(bool(causal))
    p.need_bwd = int(bool(need_bwd))
    if max_iter is not None:
        p.max_iter = int(max_iter)
    if tol is not None:
        p.tol = float(tol)
    return p


_memory = {}  # total memory of each device, a constant of the device
_held = {}    # bytes of the element lists that live Residuals hold on each device
_held_lock = threading.RLock()


def _lists_limit(device) -> int:
    """The most that the element lists of all Residuals of a device take
    together: a sixteenth of its memory."""
    if device.type != "cuda":
        return 1 << 30
    if device.index not in _memory:
        _memory[device.index] = torch.cuda.get_device_properties(device).total_memory
    return _memory[device.index] // 16


class _Claim:
    """`nbytes` of a device's share for element lists, given back when this
    object goes.  Saved and copied objects hold none."""

    def __init__(self, index, nbytes):
        self.index, self.nbytes = index, nbytes

    def __del__(self, lock=_held_lock, held=_held):  # (module globals may be gone at exit)
        with lock:
            held[self.index] -= self.nbytes

    def __reduce__(self):
        return type(None), ()


def _claim(device, nbytes):
    """A _Claim, or None where the limit would be passed."""
    limit = _lists_limit(device)
    with _held_lock:
        if _held.get(device.index, 0) + nbytes > limit:
            return None
        _held[device.index] = _held.get(device.index, 0) + nbytes
    return _Claim(device.index, nbytes)


def _lists_size(shape, params, least) -> int:
    """Bytes of the element lists, or 0: from `least` keys on (a quarter of
    that for fp32, whose products take longer), since the sort and the list
    kernel of the backward are launches of their own, and few blocks of a short
    sequence are listed."""
    if shape.seqlen <= (least if shape.dtype == EA_BF16 else least // 4):
        return 0
    return entmax_attn_lists_bytes(shape, params)


def _bytes_or_none(nbytes, device):
    try:
        return torch.empty(nbytes, dtype=torch.uint8, device=device)
    except torch.OutOfMemoryError:
        return None


# Measured, in us, with lists against without: B64 H16 n128 d64 alpha 1.5
# c = 1 150 against 140 (no block listed), B1 H1 n256 fp32 inference 26 against
# 38; the no-mask mode collects its lists in a K pass more: B1 H2 n128 56
# against 44, B1 H16 n4096 d128 670 against 1040.
LISTS_FROM, DENSE_LISTS_FROM = 256, 1024


class Residuals:
    """Device buffers (torch tensors) that the forward fills and the backward
    reads, sized by entmax_attn_sizes: tau, o2, tau_lo (fp32 inputs: the low
    part of tau), lists (the element lists, see entmax_attn_fwd_lists; 582 bytes
    a row, which the backward reads; None with lists=False, where they would
    pass a sixteenth of the device's memory together with those of every other
    live Residuals, or where there is no memory for them: forward and backward
    then run without them), and
    block_mask, q_count, q_index, k_count, k_index and stats ([0]: K passes the
    solver streamed, [1]: its evaluations, per query block).

    The last six are parts of one allocation, made into tensors where they are
    asked for: ten allocations and views per forward took longer on the host
    than the kernels of a short sequence on the GPU (a training step at B1 H2
    n128: 79 us of host time with them, most of them never looked at)."""

    lists, _tables, _parts, _kept = None, None, {}, None  # objects that were saved with a tensor per table

    def __init__(self, shape: Shape, params: Params, device, with_stats: bool = True, lists: bool = True):
        z = entmax_attn_sizes(shape, params)
        BH, n, d = shape.batch * shape.heads, shape.seqlen, shape.head_dim
        T = (n + 63) // 64
        self.shape, self.params, self.sizes = shape, params, z
        self.tau = torch.empty((BH, n), dtype=torch.float32, device=device)
        self.o2 = (torch.empty((BH, n, d), dtype=torch.float32, device=device)
                   if params.need_bwd else None)
        self.tau_lo = (torch.empty((BH, n), dtype=torch.float32, device=device)
                       if z.tau_lo else None)
        nbytes = _lists_size(shape, params, LISTS_FROM) if lists else 0
        self._share = _claim(self.tau.device, nbytes) if nbytes else None
        self.lists = _bytes_or_none(nbytes, device) if self._share else None
        at, parts = 0, {}
        for name, nbytes, dims in (
                ("q_index", z.q_index, (BH, T, T)), ("k_index", z.k_index, (BH, T, T)),
                ("q_count", z.q_count, (BH, T)), ("k_count", z.k_count, (BH, T)),
                ("stats", z.stats, (2, BH, T)), ("block_mask", z.block_mask, (BH, T, T))):
            parts[name] = (at, nbytes, dims)
            at += (nbytes + 255) // 256 * 256
        self._parts = parts
        self._tables = torch.empty(at, dtype=torch.uint8, device=device)
        if not with_stats:
            self.stats = None

    def __getattr__(self, name):  # a part that is not a tensor yet
        part = self._parts.get(name)
        if part is None:
            raise AttributeError("Residuals has no attribute %r" % name)
        at, nbytes, dims = part
        t = self._tables[at:at + nbytes]
        if name != "block_mask":
            t = t.view(torch.int32)
        t = t.view(dims)
        self.__dict__[name] = t
        return t

    def ptrs(self) -> ResidualPtrs:
        own = self.__dict__
        base = self._tables.data_ptr() if self._parts else 0

        def f(name):
            if name in own:
                return None if own[name] is None else own[name].data_ptr()
            return base + self._parts[name][0]

        p = ResidualPtrs(*map(f, ("tau", "o2", "block_mask", "q_count", "q_index", "k_count",
                                  "k_index", "stats", "tau_lo")))
        if self.lists is not None:
            p.lists, p.lists_bytes = self.lists.data_ptr(), self.lists.numel()
            p.lists_shape = _dims(self.shape)
            p.owner = self
        return p

    def keep_workspace(self, make=True):
        """The buffer that entmax_attn_bwd_noalloc sorts the lists in, held from
        the first call on; None where there is none and `make` is false, or no
        memory for it."""
        if self._kept is None and make and self.lists is not None:
            self._kept = _bytes_or_none(entmax_attn_bwd_lists_workspace(self.shape, self.params),
                                        self.lists.device)
        return self._kept


def _stream_handle(device):
    return torch._C._cuda_getCurrentRawStream(device.index)  # current_stream without its object


# ------------------------------------------------------ argument checks
#
# The C ABI takes bare device pointers and no sizes for the residual buffers,
# so a tensor of the wrong shape, dtype or device would make the kernels read
# or write past its end.  Every tensor is checked here before any call.

def _need(t, name, shape, dtype, device=None):
    """Raises ValueError unless t is a contiguous tensor of this shape and
    dtype (and, given device, on that device).  Whether that device is a GPU
    is checked once per call by _on_gpu, after every tensor's shape."""
    if not isinstance(t, torch.Tensor):
        raise ValueError("%s must be a torch tensor" % name)
    if tuple(t.shape) != tuple(shape):
        raise ValueError("%s has shape %s, expected %s" % (name, tuple(t.shape), tuple(shape)))
    if t.dtype != dtype:
        raise ValueError("%s has dtype %s, expected %s" % (name, t.dtype, dtype))
    if not t.is_contiguous():
        raise ValueError("%s must be contiguous" % name)
    if device is not None and t.device != device:
        raise ValueError("%s is on %s, expected %s" % (name, t.device, device))


def _on_gpu(device):
    if device is None or device.type != "cuda":
        raise ValueError("tensors must be on a GPU device, not %s" % device)


def _torch_dtype(shape: Shape):
    return torch.bfloat16 if shape.dtype == EA_BF16 else torch.float32


def _check_qkv(names_tensors, shape: Shape):
    """q, k, v (and dO) against one shape: [B, H, n, d] in the shape's dtype,
    all on the device of the first."""
    dims = (shape.batch, shape.heads, shape.seqlen, shape.head_dim)
    dev = names_tensors[0][1].device if isinstance(names_tensors[0][1], torch.Tensor) else None
    for name, t in names_tensors:
        _need(t, name, dims, _torch_dtype(shape), dev)
    return dev


def _same_shape(a: Shape, b: Shape) -> bool:
    return all(getattr(a, f) == getattr(b, f) for f, _ in Shape._fields_)


def _check_residuals(res, shape: Shape, device, need_o2: bool):
    if not isinstance(res, Residuals):
        raise ValueError("res must be the Residuals of a forward call")
    if not _same_shape(res.shape, shape):
        raise ValueError("res was sized for a different shape or dtype")
    BH, n, d = shape.batch * shape.heads, shape.seqlen, shape.head_dim
    T = (n + 63) // 64
    _need(res.tau, "res.tau", (BH, n), torch.float32, device)
    if need_o2:
        if res.o2 is None:
            raise ValueError("res has no o2 (forward ran with need_bwd=False)")
        _need(res.o2, "res.o2", (BH, n, d), torch.float32, device)
    # the tables that are still parts of one buffer have their sizes from it
    if res._parts:
        _need(res._tables, "res", res._tables.shape, torch.uint8, device)
    own = res.__dict__
    for name, dims, dtype in (("block_mask", (BH, T, T), torch.uint8), ("q_count", (BH, T), torch.int32),
                              ("q_index", (BH, T, T), torch.int32), ("k_count", (BH, T), torch.int32),
                              ("k_index", (BH, T, T), torch.int32), ("stats", (2, BH, T), torch.int32)):
        if name in own and not (name == "stats" and own[name] is None):
            _need(own[name], "res." + name, dims, dtype, device)
    if shape.dtype == EA_F32:
        _need(res.tau_lo, "res.tau_lo", (BH, n), torch.float32, device)
    if res.lists is not None:
        _check_bytes(res.lists, "res.lists", entmax_attn_lists_bytes(shape, res.params), device)


def _check_bytes(ws, name, need_bytes, device):
    if not isinstance(ws, torch.Tensor) or not ws.is_contiguous():
        raise ValueError("%s must be a contiguous tensor" % name)
    if ws.numel() * ws.element_size() < need_bytes:
        raise ValueError("%s holds %d bytes, needs %d" % (
            name, ws.numel() * ws.element_size(), need_bytes))
    if ws.device != device:
        raise ValueError("%s must be on %s" % (name, device))


def backward_workspace(res: Residuals, device):
    """A device buffer for the workspace of backward: delta, and room to sort
    the element lists where res has them (without that room, as in a buffer of
    sizes.ws_bwd bytes, the backward does not use them)."""
    if res.lists is not None:
        ws = _bytes_or_none(entmax_attn_bwd_lists_workspace(res.shape, res.params), device)
        if ws is not None:
            return ws
    return torch.empty(max(res.sizes.ws_bwd, 16), dtype=torch.uint8, device=device)


def forward_workspace(res: Residuals, device):
    """A device buffer of sizes.ws_fwd bytes for the solver's candidate cache."""
    return torch.empty(max(res.sizes.ws_fwd, 16), dtype=torch.uint8, device=device)


def forward(q, k, v, alpha=1.5, scale=None, causal=False, need_bwd=True, max_iter=None,
            tol=None, out=None, res: Residuals | None = None, workspace=None, lists=True):
    """O and the residuals for Q, K, V ([B, H, n, d] bf16/fp32 CUDA tensors).

    workspace: a uint8 device tensor for the solver's candidate cache (None
    allocates sizes.ws_fwd bytes; False runs the solver without the cache).
    lists: whether new residuals hold element lists (see Residuals)."""
    shape = make_shape(q)
    dev = _check_qkv([("q", q), ("k", k), ("v", v)], shape)
    params = make_params(alpha, scale, causal, need_bwd, max_iter, tol, head_dim=q.shape[-1])
    if res is None:
        res = Residuals(shape, params, q.device, lists=lists)
    else:
        _check_residuals(res, shape, dev, bool(need_bwd))
    if out is None:
        out = torch.empty_like(q)
    else:
        _need(out, "out", q.shape, q.dtype, dev)
    if workspace is not None and workspace is not False:
        _check_bytes(workspace, "workspace", 0, dev)
    _on_gpu(dev)
    rp = res.ptrs()
    if workspace is None:
        workspace = forward_workspace(res, q.device)
    ws_ptr, ws_bytes = (None, 0) if workspace is False else (workspace.data_ptr(),
                                                            workspace.numel() * workspace.element_size())
    _check(entmax_attn_fwd(shape, params, q.data_ptr(), k.data_ptr(), v.data_ptr(),
                           out.data_ptr(), rp, ws_ptr, ws_bytes, _stream_handle(q.device)),
           "entmax_attn_fwd")
    res.params = params
    return out, res


def backward(q, k, v, dout, res: Residuals, dq=None, dk=None, dv=None, workspace=None):
    """(dQ, dK, dV) in fp32 for the loss sum(dO * O) of the forward that filled res.

    workspace: a device tensor of at least sizes.ws_bwd bytes; to keep one from
    call to call, take it from backward_workspace."""
    shape = make_shape(q)
    dev = _check_qkv([("q", q), ("k", k), ("v", v), ("dout", dout)], shape)
    _check_residuals(res, shape, dev, True)
    if not res.params.need_bwd:
        raise ValueError("res comes from a forward with need_bwd=False")
    mk = lambda t: t if t is not None else torch.empty(q.shape, dtype=torch.float32, device=q.device)
    dq, dk, dv = mk(dq), mk(dk), mk(dv)
    for name, t in (("dq", dq), ("dk", dk), ("dv", dv)):
        _need(t, name, q.shape, torch.float32, dev)
    if workspace is None:
        workspace = backward_workspace(res, q.device)
    else:
        _check_bytes(workspace, "workspace", res.sizes.ws_bwd, dev)
    _on_gpu(dev)
    rp = res.ptrs()
    _check(entmax_attn_bwd(shape, res.params, q.data_ptr(), k.data_ptr(), v.data_ptr(),
                           dout.data_ptr(), rp, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(),
                           workspace.data_ptr(), workspace.numel() * workspace.element_size(),
                           _stream_handle(q.device)),
           "entmax_attn_bwd")
    return dq, dk, dv


# ------------------------------------------------------- row-wise entmax

def entmax_rows_fwd(rows, n, dtype, params, s, p, tau, stream):
    return _lib.entmax_rows_fwd(rows, n, dtype, ctypes.byref(params), s, p, tau, stream)


def entmax_rows_bwd(rows, n, dtype, params, s, tau, dp, ds, stream):
    return _lib.entmax_rows_bwd(rows, n, dtype, ctypes.byref(params), s, tau, dp, ds, stream)


def _row_params(alpha, scale, max_iter, tol):
    p = default_params()
    p.alpha, p.scale, p.causal, p.need_bwd = float(alpha), float(scale), 0, 0
    if max_iter is not None:
        p.max_iter = int(max_iter)
    if tol is not None:
        p.tol = float(tol)
    return p


def rows_forward(s, alpha=1.5, scale=1.0, max_iter=None, tol=None):
    """(p, tau): alpha-entmax of each row of s ([..., n] bf16/fp32 device tensor)."""
    if not s.is_cuda or not s.is_contiguous() or s.dtype not in (torch.bfloat16, torch.float32):
        raise ValueError("s must be a contiguous bf16 or fp32 device tensor")
    n = s.shape[-1]
    rows = s.numel() // n
    p = torch.empty(s.shape, dtype=torch.float32, device=s.device)
    tau = torch.empty(s.shape[:-1], dtype=torch.float32, device=s.device)
    params = _row_params(alpha, scale, max_iter, tol)
    _check(entmax_rows_fwd(rows, n, EA_BF16 if s.dtype == torch.bfloat16 else EA_F32, params,
                           s.data_ptr(), p.data_ptr(), tau.data_ptr(), _stream_handle(s.device)),
           "entmax_rows_fwd")
    return p, tau


def rows_backward(s, tau, dp, alpha=1.5, scale=1.0):
    """Gradient of sum(dp * p) with respect to s, for (p, tau) = rows_forward(s)."""
    if not isinstance(s, torch.Tensor) or s.dtype not in (torch.bfloat16, torch.float32):
        raise ValueError("s must be a bf16 or fp32 tensor")
    _need(s, "s", s.shape, s.dtype)
    n = s.shape[-1]
    rows = s.numel() // n
    _need(dp, "dp", s.shape, torch.float32, s.device)
    _need(tau, "tau", s.shape[:-1], torch.float32, s.device)
    _on_gpu(s.device)
    ds = torch.empty(s.shape, dtype=torch.float32, device=s.device)
    params = _row_params(alpha, scale, None, None)
    _check(entmax_rows_bwd(rows, n, EA_BF16 if s.dtype == torch.bfloat16 else EA_F32, params,
                           s.data_ptr(), tau.data_ptr(), dp.data_ptr(), ds.data_ptr(),
                           _stream_handle(s.device)), "entmax_rows_bwd")
    return ds


# ---------------------------------------------------------- no-mask mode

def _dense_backward_pays(shape, params) -> bool:
    """Whether the no-mask backward takes long enough by products (120 us and
    more; about 3.5 us per block of keys that a workgroup walks, or 215 blocks
    of 64 x 64 x 64 a microsecond, 1.6 times that with a general alpha) for the launches that look for sparse heads
    (15 us) and what those may gain: B4 H2 n1920 d64 causal, 88 us by products
    and 75 with lists at c = 12, is left out, B1 H8 n2431 d128 (181 us, 100 with
    lists) is not.  fp32 products take 16 times as long."""
    T = (shape.seqlen + 63) // 64
    blocks = shape.batch * shape.heads * T * (T + 1 if params.causal else 2 * T) // 2 * shape.head_dim // 64
    us = max(3.5 * T, blocks / 215) * (1.0 if params.alpha in (1.25, 1.5, 2.0) else 1.6)
    return shape.dtype == EA_F32 or us >= 120


def _scratch_lists(shape, params, device, lists):
    """Element lists for one call of the no-mask mode: (tensor or None, pointer, bytes)."""
    nbytes = _lists_size(shape, params, DENSE_LISTS_FROM) if lists else 0
    t = _bytes_or_none(nbytes, device) if 0 < nbytes <= _lists_limit(device) else None
    return (None, None, 0) if t is None else (t, t.data_ptr(), nbytes)


def forward_dense(q, k, v, alpha=1.5, scale=None, causal=False, need_bwd=True, max_iter=None,
                  tol=None, workspace=None, lists=True):
    """(O, tau, O2 or None, tau_lo or None) without block mask or tables
    (Algorithm 2 as written); tau_lo, the threshold's low part, exists for fp32
    inputs and goes back into backward_dense.  lists: whether the call may take
    scratch for element lists (582 bytes a row; backward_dense 1.2 KB)."""
    shape = make_shape(q)
    dev = _check_qkv([("q", q), ("k", k), ("v", v)], shape)
    _on_gpu(dev)
    params = make_params(alpha, scale, causal, need_bwd, max_iter, tol, head_dim=q.shape[-1])
    B, H, n, d = q.shape
    o = torch.empty_like(q)
    tau = torch.empty((B * H, n), dtype=torch.float32, device=q.device)
    tau_lo = torch.empty_like(tau) if q.dtype == torch.float32 else None
    o2 = torch.empty(q.shape, dtype=torch.float32, device=q.device) if need_bwd else None
    z = entmax_attn_sizes(shape, params)
    if workspace is None:
        workspace = torch.empty(max(z.ws_fwd, 16), dtype=torch.uint8, device=q.device)
    elif workspace is not False:
        _check_bytes(workspace, "workspace", 0, dev)
    _on_gpu(dev)
    ws_ptr, ws_bytes = (None, 0) if workspace is False else (workspace.data_ptr(),
                                                            workspace.numel() * workspace.element_size())
    _lists, lists_ptr, lists_bytes = _scratch_lists(shape, params, q.device, lists)
    _check(_lib.entmax_attn_fwd_dense_lists(
        ctypes.byref(shape), ctypes.byref(params), q.data_ptr(), k.data_ptr(), v.data_ptr(),
        o.data_ptr(), tau.data_ptr(), tau_lo.data_ptr() if tau_lo is not None else None,
        o2.data_ptr() if o2 is not None else None, lists_ptr, lists_bytes, ws_ptr, ws_bytes,
        _stream_handle(q.device)), "entmax_attn_fwd_dense")
    return o, tau, o2, tau_lo


def backward_dense(q, k, v, dout, tau, o2, alpha=1.5, scale=None, causal=False, tau_lo=None,
                   lists=True):
    """(dQ, dK, dV) in fp32 for the no-mask forward that produced tau, o2 and
    (fp32 inputs) tau_lo.  lists: as for forward_dense."""
    shape = make_shape(q)
    dev = _check_qkv([("q", q), ("k", k), ("v", v), ("dout", dout)], shape)
    B, H, n, d = q.shape
    _need(tau, "tau", (B * H, n), torch.float32, dev)
    _need(o2, "o2", q.shape, torch.float32, dev)
    if q.dtype == torch.float32:
        if tau_lo is None:
            raise ValueError("backward_dense: fp32 inputs need the forward's tau_lo")
        _need(tau_lo, "tau_lo", (B * H, n), torch.float32, dev)
    _on_gpu(dev)
    params = make_params(alpha, scale, causal, True, None, None, head_dim=q.shape[-1])
    mk = lambda: torch.empty(q.shape, dtype=torch.float32, device=q.device)
    dq, dk, dv = mk(), mk(), mk()
    _lists, lists_ptr, lists_bytes = _scratch_lists(shape, params, q.device,
                                                    lists and _dense_backward_pays(shape, params))
    ws = _bytes_or_none(entmax_attn_bwd_lists_workspace(shape, params), q.device) if lists_ptr else None
    if ws is None:
        ws = torch.empty(max(entmax_attn_sizes(shape, params).ws_bwd, 16), dtype=torch.uint8, device=q.device)
    _check(_lib.entmax_attn_bwd_dense_lists(
        ctypes.byref(shape), ctypes.byref(params), q.data_ptr(), k.data_ptr(), v.data_ptr(),
        dout.data_ptr(), tau.data_ptr(), tau_lo.data_ptr() if q.dtype == torch.float32 else None,
        o2.data_ptr(), lists_ptr, lists_bytes, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(),
        ws.data_ptr(), ws.numel(), _stream_handle(q.device)), "entmax_attn_bwd_dense")
    return dq, dk, dv

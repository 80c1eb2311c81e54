"""Thin ctypes binding over libcox.so (the C ABI declared in include/cox.h).

Every function here only marshals arguments: it checks tensor dtype, device
and contiguity, allocates outputs and workspaces with torch (device memory
plumbing), passes raw device pointers and torch's current HIP stream to the
C entry point of the same name, and raises ``CoxError`` on a nonzero
status.  All computation happens in the library's HIP kernels; there is no
CPU fallback.  If libcox.so has not been built, loading raises.

The ordinary calls first try the same marshalling in native code
(csrc/bind.cpp, built as _coxbind.so): plain contiguous tensors, the default
schedule and a cached workspace that is large enough.  It declines anything
else, and the Python code below does the work; so it does, with a warning, if
_coxbind.so has not been built or does not load.
"""
import ctypes as C
import importlib.util
import os
import warnings

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libcox.so")
_BIND_PATH = os.path.join(_HERE, "_coxbind.so")

I32, U32, F32, BF16 = 0, 1, 2, 3
PLAIN, TWOSUM = 0, 1
SHFL_IDX, SHFL_UP, SHFL_DOWN, SHFL_XOR = 0, 1, 2, 3
OP_REDUCE, OP_DOT, OP_SCAN, OP_COMPACT, OP_SEGMENTED, OP_CG, OP_GRID_EXCHANGE, OP_INTEGRAL_IMAGE = range(8)
CG_CONVERGED, CG_MAX_ITER, CG_BREAKDOWN, CG_ABORTED = 0, 1, 2, 3

ERR_TIMEOUT = 7


class CoxError(RuntimeError):
    def __init__(self, code, what, lib=None):
        msg = f"{what}: status {code}"
        if lib is not None:
            msg += f" ({lib.cox_status_string(code).decode()})"
            if code == 4:
                msg += f", hipError {lib.cox_last_hip_error()}"
        super().__init__(msg)
        self.code = code


class cox_cfg(C.Structure):
    _fields_ = [("items_per_lane", C.c_int32), ("warps_per_block", C.c_int32),
                ("grid_blocks", C.c_int32), ("reserved", C.c_int32)]


_lib = None

_P, _I64, _I, _SZ = C.c_void_p, C.c_int64, C.c_int, C.c_size_t
_SIGS = {
    "cox_status_string": (C.c_char_p, [_I]),
    "cox_last_hip_error": (_I, []),
    "cox_version": (_I, []),
    "cox_default_cfg": (_I, [_I, _I, C.POINTER(cox_cfg)]),
    "cox_workspace_bytes": (_SZ, [_I, _I, _I64, _I64, C.POINTER(cox_cfg)]),
    "cox_workspace_init": (_I, [_P, _SZ, _P]),
    "cox_workspace_status": (_I, [_P, _P]),
    "cox_warp_shfl": (_I, [_P, _P, _I64, _I, C.c_int32, _P, _I, _P, _P]),
    "cox_warp_vote": (_I, [_P, _P, _I64, _P, _P, _P]),
    "cox_tile_vote": (_I, [_P, _I64, _I, _P, _P, _P]),
    "cox_warp_reduce_blocks_i32": (_I, [_P, _I64, _P, _P, _P]),
    "cox_warp_reduce": (_I, [_P, _I, _I64, _I, C.POINTER(cox_cfg), _P, _P, _P, _SZ, _P]),
    "cox_warp_dot": (_I, [_P, _P, _I, _I64, _I, C.POINTER(cox_cfg), _P, _P, _P, _SZ, _P]),
    "cox_warp_reduce_away": (_I, [_P, _P, _I, _I64, _I, C.POINTER(cox_cfg), _P, _P, C.c_int32, C.c_uint32, _P, _SZ,
                                  _P]),
    "cox_warp_scan": (_I, [_P, _P, _I64, C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_warp_scan_noalloc": (_I, [_P, _P, _I64, C.POINTER(cox_cfg), _P, _P]),
    "cox_ballot_compact": (_I, [_P, _I64, _P, _P, C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_warp_scan_away": (_I, [_P, _P, _I64, C.c_int32, C.c_uint32, _P, _SZ, _P]),
    "cox_ballot_compact_away": (_I, [_P, _I64, _P, _P, C.c_int32, C.c_uint32, _P, _SZ, _P]),
    "cox_tile_sort": (_I, [_P, _P, _I64, _I, C.POINTER(cox_cfg), _P]),
    "cox_tile_sort_kv": (_I, [_P, _P, _P, _P, _I64, _I, C.POINTER(cox_cfg), _P]),
    "cox_tile_reduce": (_I, [_P, _I64, _I, _P, _P]),
    "cox_warp_masked": (_I, [_P, _I64, _I, _P, _P, _P]),
    "cox_warp_dynamic": (_I, [_P, _I64, _I, _P, _P, _P, _P, _P, _P]),
    "cox_segmented": (_I, [_P, _I, _P, _I64, _I64, _P, _P, _P, _P, _I, C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_segmented_reduce": (_I, [_P, _I, _P, _I64, _I64, _P, C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_segmented_scan": (_I, [_P, _I, _P, _I64, _I64, _P, C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_segmented_compact": (_I, [_P, _I, _P, _I64, _I64, _P, _P, C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_segmented_fused": (_I, [_P, _I, _P, _I64, _I64, _P, _P, _P, _P, C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_segmented_per_segment": (_I, [_P, _I, _P, _P, _I64, _I64, _P, _P, _P, _P, C.POINTER(cox_cfg), _P,
                                       _SZ, _P]),
    "cox_plan_segmented": (_I, [_P, _I, _P, _I64, _I64, _P, _P, _P, _P, _I, C.POINTER(cox_cfg), _I, _P, _SZ, _P,
                                C.POINTER(C.c_void_p)]),
    "cox_plan_execute": (_I, [_P, _P]),
    "cox_plan_get_cfg": (_I, [_P, C.POINTER(cox_cfg)]),
    "cox_plan_destroy": (_I, [_P]),
    "cox_integral_image": (_I, [_P, _I64, _I64, _P, _P, _SZ, _P]),
    "cox_grid_capacity": (_I, [C.POINTER(C.c_int32)]),
    "cox_grid_exchange": (_I, [C.c_int32, C.c_int32, _P, _P, _SZ, _P]),
    "cox_grid_exchange_absent": (_I, [C.c_int32, C.c_int32, C.c_int32, C.c_uint32, _P, _P, _SZ, _P]),
    "cox_cg_solve": (_I, [_P, _P, _P, _I64, _I64, _P, _P, C.c_int32, C.c_double, _P, _P, C.POINTER(cox_cfg), _P,
                          _SZ, _P]),
    "cox_cg_solve_per_phase": (_I, [_P, _P, _P, _I64, _I64, _P, _P, C.c_int32, C.c_double, _P, _P,
                                    C.POINTER(cox_cfg), _P, _SZ, _P]),
    "cox_stream_read": (_I, [_P, _SZ, _P, C.c_int32, _P]),
    "cox_stream_copy": (_I, [_P, _P, _SZ, C.c_int32, _P]),
}


# What a small call costs is the host's work per call: a launch takes about
# 3 us, a kernel on a small input 3 to 6 us.  So pointers and streams are plain
# integers, the stream is read through torch's raw-handle query (0.2 us;
# torch.cuda.current_stream() builds a Stream object, 2.9 us), the library's
# default schedules, which are constants, are asked for once, and ordinary
# calls allocate and call in native code.  Python calls of block reduce (2^20),
# float32 sum (65,613) and 32-key sort (2^22 + 17): 10.0 / 13.0 / 8.9 us before,
# 5.4 / 6.1 / 5.7 us now.
_native = None


class _NoNative:
    """Stands in for _coxbind.so: declines every call, so that the Python code
    makes it."""

    def __getattr__(self, name):
        return lambda *args: None


def _load_native(L):
    try:
        spec = importlib.util.spec_from_file_location("_coxbind", _BIND_PATH)
        native = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(native)
    except (ImportError, OSError) as e:
        warnings.warn(f"{_BIND_PATH} does not load ({e}): calls cost some microseconds more; "
                      "build it with __graft_entry__.build()")
        return _NoNative()
    native.init(*(C.cast(getattr(L, name), C.c_void_p).value for name in (
        "cox_warp_reduce_blocks_i32", "cox_warp_reduce", "cox_warp_dot", "cox_warp_scan", "cox_ballot_compact",
        "cox_tile_sort", "cox_tile_reduce", "cox_warp_masked", "cox_segmented", "cox_integral_image")))
    return native


def lib():
    """Loads libcox.so once; raises if it has not been built."""
    global _lib, _native
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with __graft_entry__.build() "
                               "(there is no CPU fallback)")
        L = C.CDLL(LIB_PATH)
        for name, (res, args) in _SIGS.items():
            f = getattr(L, name)
            f.restype = res
            f.argtypes = args
        _native = _load_native(L)
        _lib = L
    return _lib


def exported_symbols():
    return sorted(_SIGS)


def _check(code, what):
    if code != 0:
        raise CoxError(code, what, lib())


ERR_WORKSPACE = 5


def _done(r, what):
    """Whether a native call's answer stands: None was declined, and a
    workspace that is too small is replaced by the Python path."""
    if type(r) is int:
        if r == ERR_WORKSPACE:
            return False
        raise CoxError(r, what, lib())
    return r is not None


def _on_gpu(x):
    """Whether the native path can be asked: x is a device tensor (and the
    library is loaded)."""
    return isinstance(x, torch.Tensor) and x.is_cuda and (_native is not None or lib() is not None)


def _cached_ws(op, x):
    """The cached workspace of this operation on tensor x's device, or None."""
    return _ws_cache.get((op, x.get_device())) if isinstance(x, torch.Tensor) else None


def _ptr(t):
    return None if t is None else t.data_ptr()


def _stream():
    """torch's current HIP stream on the current device, as an integer."""
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())


def _need(t, dtype, name):
    if isinstance(t, torch.Tensor) and t.is_cuda and t.dtype == dtype and t.is_contiguous():
        return
    if not isinstance(t, torch.Tensor) or not t.is_cuda:
        raise TypeError(f"{name} must be a CUDA (HIP) tensor")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    raise ValueError(f"{name} must be contiguous")


_CODES = {torch.int32: I32, torch.float32: F32, torch.bfloat16: BF16}


def _dtype_code(t):
    code = _CODES.get(t.dtype)
    if code is None:
        raise TypeError(f"unsupported dtype {t.dtype}")
    return code


def make_cfg(items_per_lane=0, warps_per_block=0, grid_blocks=0):
    return cox_cfg(int(items_per_lane), int(warps_per_block), int(grid_blocks), 0)


def _cfgp(cfg):
    if cfg is None:
        return None
    if isinstance(cfg, (tuple, list)):
        cfg = make_cfg(*cfg)
    return C.byref(cfg)


_default_cfgs = {}


def default_cfg(op, dtype=I32):
    d = _default_cfgs.get((op, dtype))
    if d is None:
        c = cox_cfg()
        _check(lib().cox_default_cfg(op, dtype, C.byref(c)), "cox_default_cfg")
        d = _default_cfgs[(op, dtype)] = (c.items_per_lane, c.warps_per_block, c.grid_blocks)
    return d


# ---------------------------------------------------------------- workspaces
class Workspace:
    """A zero-initialised device workspace owned by the caller."""

    def __init__(self, nbytes, device=None):
        nbytes = max(256, (int(nbytes) + 255) // 256 * 256)
        self.tensor = torch.empty(nbytes, dtype=torch.uint8, device=device or "cuda")
        self.nbytes = nbytes
        self.ptr = self.tensor.data_ptr()
        _check(lib().cox_workspace_init(_ptr(self.tensor), nbytes, _stream()), "cox_workspace_init")

    def status(self):
        """Synchronises the stream; raises CoxError(COX_ERR_TIMEOUT) if a
        bounded cross-block wait gave up since the last check."""
        _check(lib().cox_workspace_status(_ptr(self.tensor), _stream()), "cox_workspace_status")


_ws_cache = {}


def workspace(op, dtype, n, nseg=0, cfg=None, device=None):
    """Per-(op, device) cached workspace large enough for this call."""
    need = lib().cox_workspace_bytes(op, dtype, int(n), int(nseg), _cfgp(cfg))
    if need == 0:
        raise CoxError(1, "cox_workspace_bytes", lib())
    if device is None:
        dev = torch.device("cuda", torch.cuda.current_device())
    else:
        dev = device if isinstance(device, torch.device) else torch.device(device)
    key = (op, dev.index)
    ws = _ws_cache.get(key)
    if ws is None or ws.nbytes < need:
        ws = Workspace(need, dev)
        _ws_cache[key] = ws
    return ws


# ---------------------------------------------------------------- entry points
def warp_shfl(v, op, arg=0, width=32, mask=None, argv=None, out=None):
    _need(v, torch.int32, "v")
    n = v.numel()
    out = torch.empty_like(v) if out is None else out
    if mask is not None:
        _need(mask, torch.int32, "mask")  # uint32 bits carried in int32
    if argv is not None:
        _need(argv, torch.int32, "argv")
    _check(lib().cox_warp_shfl(_ptr(v), _ptr(out), n, int(op), int(arg), _ptr(argv), int(width),
                               _ptr(mask), _stream()), "cox_warp_shfl")
    return out


def warp_vote(pred, mask=None):
    _need(pred, torch.int32, "pred")
    g = pred.numel() // 32
    bal = torch.zeros(g, dtype=torch.int32, device=pred.device)
    aa = torch.zeros(g, dtype=torch.int32, device=pred.device)
    if mask is not None:
        _need(mask, torch.int32, "mask")
    _check(lib().cox_warp_vote(_ptr(pred), _ptr(mask), pred.numel(), _ptr(bal), _ptr(aa), _stream()),
           "cox_warp_vote")
    return bal, aa


def tile_vote(pred, tile):
    """Per tile of `tile` lanes: (T-bit ballot, any | all << 1) as int32
    device tensors of n / tile entries."""
    _need(pred, torch.int32, "pred")
    g = pred.numel() // tile if tile > 0 else 0
    bal = torch.zeros(g, dtype=torch.int32, device=pred.device)
    aa = torch.zeros(g, dtype=torch.int32, device=pred.device)
    _check(lib().cox_tile_vote(_ptr(pred), pred.numel(), int(tile), _ptr(bal), _ptr(aa), _stream()),
           "cox_tile_vote")
    return bal, aa


def warp_reduce_blocks_i32(x, block_sums=None, warp_pos_count=None):
    if _on_gpu(x):
        r = _native.reduce_blocks(x, block_sums, warp_pos_count, _stream())
        if _done(r, "cox_warp_reduce_blocks_i32"):
            return r
    _need(x, torch.int32, "x")
    n = x.numel()
    if block_sums is None:
        block_sums = torch.empty((n + 255) // 256, dtype=torch.int32, device=x.device)
    if warp_pos_count is None:
        warp_pos_count = torch.empty((n + 31) // 32, dtype=torch.int32, device=x.device)
    _check(lib().cox_warp_reduce_blocks_i32(_ptr(x), n, _ptr(block_sums), _ptr(warp_pos_count), _stream()),
           "cox_warp_reduce_blocks_i32")
    return block_sums, warp_pos_count


def _kw(cfg):
    if cfg is None:
        return 0, 0
    if isinstance(cfg, (tuple, list)):
        return (tuple(cfg) + (0, 0))[:2]
    return cfg.items_per_lane, cfg.warps_per_block


def _nchunks(n, cfg, op, dt):
    k, W = _kw(cfg)
    dk, dW, _ = default_cfg(op, dt)
    k, W = k or dk, W or dW
    S = 32 * W * k
    return (n + S - 1) // S


def _reduce_native(op, x, y, acc, partials):
    ws = _cached_ws(op, x)
    code = _CODES.get(x.dtype) if ws is not None else None
    if code is None or acc not in (PLAIN, TWOSUM):
        return None
    k, W, _ = default_cfg(op, code)
    return _native.reduce(x, y, int(acc), 32 * k * W if partials else 0, ws.ptr, ws.nbytes, _stream())


def warp_reduce(x, acc=PLAIN, cfg=None, partials=True, total=None, partials_out=None):
    """Returns (total, chunk_partials or None) as device tensors: total is
    int64 for int32 input, float64 otherwise."""
    if cfg is None and total is None and partials_out is None:
        r = _reduce_native(OP_REDUCE, x, None, acc, partials)
        if _done(r, "cox_warp_reduce"):
            return r
    dt = _dtype_code(x)
    _need(x, x.dtype, "x")
    n = x.numel()
    if total is None:
        total = torch.empty(1, dtype=torch.int64 if dt == I32 else torch.float64, device=x.device)
    part = partials_out
    if part is None and partials:
        nch = _nchunks(n, cfg, OP_REDUCE, dt)
        shape = (nch, 2) if acc == TWOSUM else (nch,)
        part = torch.empty(shape, dtype=torch.int32 if dt == I32 else torch.float32, device=x.device)
    ws = workspace(OP_REDUCE, dt, n, cfg=cfg, device=x.device)
    _check(lib().cox_warp_reduce(_ptr(x), dt, n, int(acc), _cfgp(cfg), _ptr(part), _ptr(total),
                                 _ptr(ws.tensor), ws.nbytes, _stream()), "cox_warp_reduce")
    return total, part


def warp_dot(a, b, acc=PLAIN, cfg=None, partials=True, total=None, partials_out=None):
    if cfg is None and total is None and partials_out is None and b is not None:
        r = _reduce_native(OP_DOT, a, b, acc, partials)
        if _done(r, "cox_warp_dot"):
            return r
    dt = _dtype_code(a)
    _need(a, a.dtype, "a")
    _need(b, a.dtype, "b")
    if a.numel() != b.numel():
        raise ValueError("a and b differ in size")
    n = a.numel()
    if total is None:
        total = torch.empty(1, dtype=torch.float64, device=a.device)
    part = partials_out
    if part is None and partials:
        nch = _nchunks(n, cfg, OP_DOT, dt)
        shape = (nch, 2) if acc == TWOSUM else (nch,)
        part = torch.empty(shape, dtype=torch.float32, device=a.device)
    ws = workspace(OP_DOT, dt, n, cfg=cfg, device=a.device)
    _check(lib().cox_warp_dot(_ptr(a), _ptr(b), dt, n, int(acc), _cfgp(cfg), _ptr(part), _ptr(total),
                              _ptr(ws.tensor), ws.nbytes, _stream()), "cox_warp_dot")
    return total, part


def warp_reduce_away(x, y=None, acc=PLAIN, cfg=None, away_block=0, polls=0):
    """warp_reduce (or warp_dot with y) with one block starting late and a
    small bound on the wait for it."""
    dt = _dtype_code(x)
    op = OP_REDUCE if y is None else OP_DOT
    _need(x, x.dtype, "x")
    if y is not None:
        _need(y, x.dtype, "y")
        if x.numel() != y.numel():
            raise ValueError("x and y differ in size")
    n = x.numel()
    integer = dt == I32
    total = torch.empty(1, dtype=torch.int64 if integer else torch.float64, device=x.device)
    nch = _nchunks(n, cfg, op, dt)
    part = torch.empty((nch, 2) if acc == TWOSUM else (nch,), dtype=torch.int32 if integer else torch.float32,
                       device=x.device)
    ws = workspace(op, dt, n, cfg=cfg, device=x.device)
    _check(lib().cox_warp_reduce_away(_ptr(x), _ptr(y), dt, n, int(acc), _cfgp(cfg), _ptr(part), _ptr(total),
                                      int(away_block), int(polls), _ptr(ws.tensor), ws.nbytes, _stream()),
           "cox_warp_reduce_away")
    return total, part


def warp_scan(x, cfg=None, out=None):
    ws = _cached_ws(OP_SCAN, x)
    if cfg is None and ws is not None:
        r = _native.scan(x, out, ws.ptr, ws.nbytes, _stream())
        if _done(r, "cox_warp_scan"):
            return r
    _need(x, torch.int32, "x")
    n = x.numel()
    y = torch.empty_like(x) if out is None else out
    ws = workspace(OP_SCAN, I32, n, cfg=cfg, device=x.device)
    _check(lib().cox_warp_scan(_ptr(x), _ptr(y), n, _cfgp(cfg), _ptr(ws.tensor), ws.nbytes, _stream()),
           "cox_warp_scan")
    return y


def warp_scan_noalloc(x, cfg=None, out=None, err=None):
    """cox_warp_scan on the library's fixed device scratch (no workspace).
    err: optional 1-element int32 device tensor receiving the wait status."""
    _need(x, torch.int32, "x")
    y = torch.empty_like(x) if out is None else out
    if err is not None:
        _need(err, torch.int32, "err")
    _check(lib().cox_warp_scan_noalloc(_ptr(x), _ptr(y), x.numel(), _cfgp(cfg), _ptr(err), _stream()),
           "cox_warp_scan_noalloc")
    return y


def ballot_compact(x, cfg=None, out=None, count=None):
    """Returns (out buffer of capacity n, count as a 1-element int64 device
    tensor); the kept elements are out[:count]."""
    ws = _cached_ws(OP_COMPACT, x)
    if cfg is None and ws is not None:
        r = _native.compact(x, out, count, ws.ptr, ws.nbytes, _stream())
        if _done(r, "cox_ballot_compact"):
            return r
    _need(x, torch.int32, "x")
    n = x.numel()
    out = torch.empty_like(x) if out is None else out
    count = torch.empty(1, dtype=torch.int64, device=x.device) if count is None else count
    ws = workspace(OP_COMPACT, I32, n, cfg=cfg, device=x.device)
    _check(lib().cox_ballot_compact(_ptr(x), n, _ptr(out), _ptr(count), _cfgp(cfg), _ptr(ws.tensor),
                                    ws.nbytes, _stream()), "cox_ballot_compact")
    return out, count


def warp_scan_away(x, away_block=0, polls=0):
    """warp_scan of a short input with one block starting late and a small
    bound on the wait for it."""
    _need(x, torch.int32, "x")
    n, y = x.numel(), torch.empty_like(x)
    ws = workspace(OP_SCAN, I32, n, device=x.device)
    _check(lib().cox_warp_scan_away(_ptr(x), _ptr(y), n, int(away_block), int(polls), _ptr(ws.tensor), ws.nbytes,
                                    _stream()), "cox_warp_scan_away")
    return y


def ballot_compact_away(x, away_block=0, polls=0):
    """ballot_compact of a short input with one block starting late and a
    small bound on the wait for it."""
    _need(x, torch.int32, "x")
    n, out = x.numel(), torch.empty_like(x)
    count = torch.empty(1, dtype=torch.int64, device=x.device)
    ws = workspace(OP_COMPACT, I32, n, device=x.device)
    _check(lib().cox_ballot_compact_away(_ptr(x), n, _ptr(out), _ptr(count), int(away_block), int(polls),
                                         _ptr(ws.tensor), ws.nbytes, _stream()), "cox_ballot_compact_away")
    return out, count


def tile_sort(keys, tile=32, cfg=None, out=None):
    """keys: int32 tensor holding uint32 bit patterns (sorted as unsigned)."""
    if cfg is None and _on_gpu(keys):
        r = _native.sort(keys, int(tile), out, _stream())
        if _done(r, "cox_tile_sort"):
            return r
    _need(keys, torch.int32, "keys")
    out = torch.empty_like(keys) if out is None else out
    _check(lib().cox_tile_sort(_ptr(keys), _ptr(out), keys.numel(), int(tile), _cfgp(cfg), _stream()),
           "cox_tile_sort")
    return out


def tile_sort_kv(keys, vals, cfg=None, out_keys=None, out_vals=None):
    """Stable sort of every 32-pair group by unsigned key (keys: int32 view
    of uint32 keys; vals: any 4-byte int32 / float32 tensor).  Returns
    (out_keys, out_vals)."""
    _need(keys, torch.int32, "keys")
    if vals.dtype not in (torch.int32, torch.float32):
        raise TypeError("vals must be a 4-byte tensor (int32 or float32)")
    _need(vals, vals.dtype, "vals")
    n = keys.numel()
    if vals.numel() != n:
        raise ValueError("keys and vals differ in size")
    out_keys = torch.empty_like(keys) if out_keys is None else out_keys
    out_vals = torch.empty_like(vals) if out_vals is None else out_vals
    _check(lib().cox_tile_sort_kv(_ptr(keys), _ptr(vals), _ptr(out_keys), _ptr(out_vals), n, 32, _cfgp(cfg),
                                  _stream()), "cox_tile_sort_kv")
    return out_keys, out_vals


def tile_reduce(x, tile, out=None):
    if type(tile) is int and _on_gpu(x):
        r = _native.tile_reduce(x, tile, out, _stream())
        if _done(r, "cox_tile_reduce"):
            return r
    _need(x, torch.int32, "x")
    n = x.numel()
    out = torch.empty((n + tile - 1) // tile, dtype=torch.int32, device=x.device) if out is None else out
    _check(lib().cox_tile_reduce(_ptr(x), n, int(tile), _ptr(out), _stream()), "cox_tile_reduce")
    return out


def warp_masked(x, density, out=None, rec=None):
    if _on_gpu(x):
        r = _native.masked(x, int(density), out, rec, _stream())
        if _done(r, "cox_warp_masked"):
            return r
    _need(x, torch.int32, "x")
    n = x.numel()
    out = torch.empty_like(x) if out is None else out
    rec = torch.empty((n // 32, 4), dtype=torch.int32, device=x.device) if rec is None else rec
    _check(lib().cox_warp_masked(_ptr(x), n, int(density), _ptr(out), _ptr(rec), _stream()),
           "cox_warp_masked")
    return out, rec


def warp_dynamic(x, density, match_any=None, rank=None, rec=None, filtered=None, count=None):
    """Dynamic groups (coalesced_threads, match_any / match_all, the six
    reduce_*_sync, warp-aggregated append).  Returns (match_any, rank,
    rec[n/32, 8], filtered (capacity n), count as a 1-element int64 device
    tensor); the members are filtered[:count]."""
    _need(x, torch.int32, "x")
    n = x.numel()
    dev = x.device
    match_any = torch.empty(n, dtype=torch.int32, device=dev) if match_any is None else match_any
    rank = torch.empty(n, dtype=torch.int32, device=dev) if rank is None else rank
    rec = torch.empty((n // 32, 8), dtype=torch.int32, device=dev) if rec is None else rec
    filtered = torch.empty_like(x) if filtered is None else filtered
    count = torch.empty(1, dtype=torch.int64, device=dev) if count is None else count
    _check(lib().cox_warp_dynamic(_ptr(x), n, int(density), _ptr(match_any), _ptr(rank), _ptr(rec), _ptr(filtered),
                                  _ptr(count), _stream()), "cox_warp_dynamic")
    return match_any, rank, rec, filtered, count


def integral_image(img, out=None):
    """Summed-area table (mod 2^32) of a uint8 device image [H, W]; returns
    an int32 tensor holding the uint32 sums."""
    ws = _ws_cache.get((OP_INTEGRAL_IMAGE, torch._C._cuda_getDevice())) if _ws_cache else None
    if ws is not None:
        r = _native.image(img, out, ws.ptr, ws.nbytes, _stream())
        if _done(r, "cox_integral_image"):
            return r
    _need(img, torch.uint8, "img")
    if img.dim() != 2:
        raise ValueError("img must be 2-D [height, width]")
    H, W = img.shape
    out = torch.empty((H, W), dtype=torch.int32, device=img.device) if out is None else out
    ws = workspace(OP_INTEGRAL_IMAGE, U32, H, W)
    _check(lib().cox_integral_image(_ptr(img), H, W, _ptr(out), _ptr(ws.tensor), ws.nbytes, _stream()),
           "cox_integral_image")
    return out


def grid_capacity():
    """Largest grid of 1024-thread blocks a cooperative launch can hold."""
    v = C.c_int32()
    _check(lib().cox_grid_capacity(C.byref(v)), "cox_grid_capacity")
    return v.value


def grid_exchange(grid_blocks, rounds, out=None):
    """Exchange kernel over a grid barrier; returns uint32 sums as an int32
    device tensor [grid_blocks, 1024].  The workspace's timeout flag is
    checked (synchronising)."""
    out = torch.empty((grid_blocks, 1024), dtype=torch.int32, device="cuda") if out is None else out
    ws = workspace(OP_GRID_EXCHANGE, U32, grid_blocks)
    _check(lib().cox_grid_exchange(int(grid_blocks), int(rounds), _ptr(out), _ptr(ws.tensor), ws.nbytes, _stream()),
           "cox_grid_exchange")
    ws.status()
    return out


def grid_exchange_absent(grid_blocks, rounds, absent_block, spin_limit):
    """The exchange kernel with one block absent from the first barrier and
    a small spin bound: returns the workspace status afterwards (expected
    COX_ERR_TIMEOUT); synchronises."""
    out = torch.empty((grid_blocks, 1024), dtype=torch.int32, device="cuda")
    ws = workspace(OP_GRID_EXCHANGE, U32, grid_blocks)
    _check(lib().cox_grid_exchange_absent(int(grid_blocks), int(rounds), int(absent_block), int(spin_limit),
                                          _ptr(out), _ptr(ws.tensor), ws.nbytes, _stream()),
           "cox_grid_exchange_absent")
    return lib().cox_workspace_status(_ptr(ws.tensor), _stream())


def cg_solve(row_ptr, col_idx, val, b, x, max_iter, tol=0.0, cfg=None, rr_hist=None, result=None,
             per_phase=False):
    """Conjugate gradient on the CSR system (row_ptr, col_idx, val) x = b,
    updating the float32 device tensor x in place (it holds x_0 on entry).
    One cooperative launch, or one launch per phase with per_phase=True.
    Returns (result, rr_hist): result = int32 device tensor {iterations,
    reason}, rr_hist = float64 device tensor [max_iter + 1]."""
    _need(row_ptr, torch.int32, "row_ptr")
    _need(col_idx, torch.int32, "col_idx")
    _need(val, torch.float32, "val")
    _need(b, torch.float32, "b")
    _need(x, torch.float32, "x")
    n, nnz = b.numel(), col_idx.numel()
    if row_ptr.numel() != n + 1 or val.numel() != nnz or x.numel() != n:
        raise CoxError(1, "cg_solve: inconsistent CSR / vector sizes")
    dev = b.device
    # every solve writes both words of the result
    result = torch.empty(2, dtype=torch.int32, device=dev) if result is None else result
    rr_hist = torch.zeros(max_iter + 1, dtype=torch.float64, device=dev) if rr_hist is None else rr_hist
    ws = workspace(OP_CG, F32, n, cfg=cfg)
    fn = lib().cox_cg_solve_per_phase if per_phase else lib().cox_cg_solve
    _check(fn(_ptr(row_ptr), _ptr(col_idx), _ptr(val), n, nnz, _ptr(b), _ptr(x), int(max_iter), float(tol),
              _ptr(result), _ptr(rr_hist), _cfgp(cfg), _ptr(ws.tensor), ws.nbytes, _stream()),
           "cox_cg_solve_per_phase" if per_phase else "cox_cg_solve")
    return result, rr_hist


def stream_read(x, sink=None, grid_blocks=0):
    """Bandwidth reference: reads every byte of tensor x once."""
    sink = torch.zeros(1, dtype=torch.int32, device=x.device) if sink is None else sink
    _check(lib().cox_stream_read(_ptr(x), x.numel() * x.element_size(), _ptr(sink), int(grid_blocks),
                                 _stream()), "cox_stream_read")
    return sink


def stream_copy(src, dst, grid_blocks=0):
    """Bandwidth reference: copies src into dst (same byte size)."""
    nb = src.numel() * src.element_size()
    if dst.numel() * dst.element_size() != nb:
        raise ValueError("size mismatch")
    _check(lib().cox_stream_copy(_ptr(src), _ptr(dst), nb, int(grid_blocks), _stream()), "cox_stream_copy")
    return dst


# ---------------------------------------------------------------- segmented
SEG_REDUCE, SEG_SCAN, SEG_COMPACT = 1, 2, 4

# the plan autotuner's candidates all use chunks of at least 4096 elements
_SEG_MIN_CHUNK_CFG = (8, 16)


def _seg_outputs(x, offsets, which, seg_total, y, out, seg_count):
    dt = _dtype_code(x)
    nseg = offsets.numel() - 1
    dev = x.device
    if which & SEG_REDUCE and seg_total is None:
        seg_total = torch.empty(nseg, dtype=torch.int64 if dt == I32 else torch.float64, device=dev)
    if which & SEG_SCAN and y is None:
        y = torch.empty_like(x)
    if which & SEG_COMPACT:
        if out is None:
            out = torch.zeros_like(x)
        if seg_count is None:
            seg_count = torch.empty(nseg, dtype=torch.int64, device=dev)
    return dt, nseg, seg_total, y, out, seg_count


def segmented(x, offsets, which=7, cfg=None, seg_total=None, y=None, out=None, seg_count=None):
    """Segmented totals / scan / compaction over CSR offsets (device int64,
    nseg + 1 entries) in one fused launch.  Returns (seg_total, y, out,
    seg_count) with None for outputs not selected by `which`."""
    ws = _cached_ws(OP_SEGMENTED, x)
    if cfg is None and ws is not None and type(which) is int:
        r = _native.segmented(x, offsets, which, seg_total, y, out, seg_count, ws.ptr, ws.nbytes, _stream())
        if _done(r, "cox_segmented"):
            return r
    _need(offsets, torch.int64, "offsets")
    if x.dtype not in (torch.int32, torch.float32):
        raise TypeError("x must be int32 or float32")
    _need(x, x.dtype, "x")
    dt, nseg, seg_total, y, out, seg_count = _seg_outputs(x, offsets, which, seg_total, y, out, seg_count)
    ws = workspace(OP_SEGMENTED, dt, x.numel(), nseg, cfg=cfg, device=x.device)
    _check(lib().cox_segmented(_ptr(x), dt, _ptr(offsets), nseg, x.numel(), _ptr(seg_total), _ptr(y), _ptr(out),
                               _ptr(seg_count), int(which), _cfgp(cfg), _ptr(ws.tensor), ws.nbytes, _stream()),
           "cox_segmented")
    return seg_total, y, out, seg_count


def segmented_per_segment(x, offsets, offsets_host, cfg=None, seg_total=None, y=None, out=None, seg_count=None):
    """Baseline: the fused kernel launched once per segment."""
    _need(offsets, torch.int64, "offsets")
    _need(x, x.dtype, "x")
    oh = offsets_host.contiguous()
    dt, nseg, seg_total, y, out, seg_count = _seg_outputs(x, offsets, 7, seg_total, y, out, seg_count)
    ws = workspace(OP_SEGMENTED, dt, x.numel(), nseg, cfg=cfg, device=x.device)
    _check(lib().cox_segmented_per_segment(_ptr(x), dt, _ptr(offsets), oh.data_ptr(), nseg, x.numel(),
                                           _ptr(seg_total), _ptr(y), _ptr(out), _ptr(seg_count), _cfgp(cfg),
                                           _ptr(ws.tensor), ws.nbytes, _stream()), "cox_segmented_per_segment")
    return seg_total, y, out, seg_count


class Plan:
    """A segmented call bound to its buffers and captured in a hipGraph;
    execute() replays it on torch's current stream."""

    def __init__(self, x, offsets, which=7, cfg=None, autotune=True, seg_total=None, y=None, out=None,
                 seg_count=None):
        _need(offsets, torch.int64, "offsets")
        _need(x, x.dtype, "x")
        dt, nseg, self.seg_total, self.y, self.out, self.seg_count = _seg_outputs(
            x, offsets, which, seg_total, y, out, seg_count)
        self.x, self.offsets = x, offsets
        wcfg = cfg if cfg is not None and any(_kw(cfg)) else _SEG_MIN_CHUNK_CFG
        nbytes = lib().cox_workspace_bytes(OP_SEGMENTED, dt, x.numel(), nseg, _cfgp(wcfg))
        forced = os.environ.get("COX_FORCE_CFG", "")
        if forced and (cfg is None or not any(_kw(cfg)[:2])):
            # the library takes this schedule when the caller gives none
            try:
                fk = [int(v) for v in forced.split(",")][:3]
                nbytes = max(nbytes, lib().cox_workspace_bytes(OP_SEGMENTED, dt, x.numel(), nseg,
                                                               _cfgp(tuple(fk[:2]))))
            except ValueError:
                pass
        self.ws = Workspace(nbytes, x.device)  # a plan owns its workspace
        h = C.c_void_p()
        _check(lib().cox_plan_segmented(_ptr(x), dt, _ptr(offsets), nseg, x.numel(), _ptr(self.seg_total),
                                        _ptr(self.y), _ptr(self.out), _ptr(self.seg_count), int(which), _cfgp(cfg),
                                        int(bool(autotune)), _ptr(self.ws.tensor), self.ws.nbytes, _stream(),
                                        C.byref(h)), "cox_plan_segmented")
        self.handle = h

    def execute(self):
        _check(lib().cox_plan_execute(self.handle, _stream()), "cox_plan_execute")
        return self.seg_total, self.y, self.out, self.seg_count

    def cfg(self):
        c = cox_cfg()
        _check(lib().cox_plan_get_cfg(self.handle, C.byref(c)), "cox_plan_get_cfg")
        return (c.items_per_lane, c.warps_per_block, c.grid_blocks)

    def close(self):
        if getattr(self, "handle", None):
            lib().cox_plan_destroy(self.handle)
            self.handle = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

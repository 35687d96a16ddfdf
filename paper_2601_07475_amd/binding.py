"""Thin ctypes binding of libarcq.so: same names as include/arcq.h and include/arcq_bench.h, argument marshalling only.

PyTorch supplies device memory and the stream; every step of the path runs in the HIP
kernels.  There is no fallback: if the library is not built, or a call fails, an exception
is raised.
"""
import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.environ.get("ARCQ_LIBRARY") or os.path.join(_HERE, "libarcq.so")   # override: a differently built copy

OK, INVALID_ARG, BAD_SHAPE, BAD_ALIGN, HIP_ERROR, WORKSPACE_TOO_SMALL = range(6)
DTYPE_F16, DTYPE_F32 = 0, 1
LAYOUT_INTERLEAVED, SCALE_ROUND_UP, RMSNORM_EXACT_SUM = 1, 2, 4
MAX_K = 65536
ROUTE_STREAM, ROUTE_KSPLIT, ROUTE_TILES, ROUTE_DIRECT = range(4)


class Route(ctypes.Structure):
    """arcq_route of arcq_bench.h."""
    _fields_ = [(n, ctypes.c_int32) for n in ("kernel", "tile_rows", "tile_cols", "runs", "ahead")]


class Rest(ctypes.Structure):
    """arcq_rest of arcq_bench.h."""
    _fields_ = [("rows", ctypes.c_int64), ("cols", ctypes.c_int64), ("route", Route)]


# every symbol include/arcq.h and include/arcq_bench.h declare: name -> (restype, argtypes)
_i64, _f32, _vp, _sz, _u32 = ctypes.c_int64, ctypes.c_float, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_uint32
SIGNATURES = {
    "arcq_version": (ctypes.c_int, []),
    "arcq_last_error": (ctypes.c_char_p, []),
    "arcq_packed_sizes": (ctypes.c_int, [_i64, _i64, _i64, ctypes.POINTER(_sz), ctypes.POINTER(_sz)]),
    "arcq_quantize_act": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _f32, _vp, _vp, _vp]),
    "arcq_rmsnorm_quantize_act": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _f32, _vp, _i64, _f32, _vp, _vp, _vp]),
    "arcq_pack_weight": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _f32, _vp, _vp, _vp]),
    "arcq_quantize_act_ex": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _f32, _u32, _vp, _vp, _vp]),
    "arcq_rmsnorm_quantize_act_ex": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _f32, _vp, _i64, _f32, _u32, _vp, _vp, _vp]),
    "arcq_pack_weight_ex": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _f32, _u32, _vp, _vp, _vp]),
    "arcq_mx_quantize_act_ex": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _u32, _vp, _vp, _vp]),
    "arcq_mx_pack_weight_ex": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _u32, _vp, _vp, _vp]),
    "arcq_mx_packed_sizes": (ctypes.c_int, [_i64, _i64, _i64, ctypes.POINTER(_sz), ctypes.POINTER(_sz)]),
    "arcq_mx_quantize_act": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _vp, _vp, _vp]),
    "arcq_mx_pack_weight": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _i64, _vp, _vp, _vp]),
    "arcq_mx_gemm": (ctypes.c_int, [_vp, _vp, _vp, _vp, _i64, _i64, _i64, _vp, ctypes.c_int, _i64, _vp]),
    "arcq_mx_gemm_workspace_size": (ctypes.c_int, [_i64, _i64, _i64, ctypes.POINTER(_sz)]),
    "arcq_mx_gemm_ws": (ctypes.c_int, [_vp, _vp, _vp, _vp, _i64, _i64, _i64, _vp, ctypes.c_int, _i64, _vp, _sz, _vp]),
    "arcq_calib_absmax": (ctypes.c_int, [_vp, _i64, _i64, _i64, _vp, _vp]),
    "arcq_calib_select": (ctypes.c_int, [_vp, _i64, _vp, _vp, _vp, _vp]),
    "arcq_gemm_workspace_size": (ctypes.c_int, [_i64, _i64, _i64, ctypes.POINTER(_sz)]),
    "arcq_gemm": (ctypes.c_int, [_vp, _vp, _f32, _vp, _vp, _f32, _i64, _i64, _i64, _vp, ctypes.c_int, _i64,
                                 _vp, _sz, _vp]),
    "arcq_gemm_noalloc": (ctypes.c_int, [_vp, _vp, _f32, _vp, _vp, _f32, _i64, _i64, _i64, _vp, ctypes.c_int, _i64, _vp]),
    "arcq_probe_mfma_f16": (ctypes.c_int, [ctypes.c_int, _vp, ctypes.POINTER(ctypes.c_double), _vp]),
    "arcq_probe_mfma_fp4": (ctypes.c_int, [ctypes.c_int, _vp, ctypes.POINTER(ctypes.c_double), _vp]),
    "arcq_probe_buffer_copy": (ctypes.c_int, [_vp, _u32, _u32, ctypes.c_int, _vp, _vp]),
    "arcq_ref_gemm_bf16": (ctypes.c_int, [_vp, _vp, _i64, _i64, _i64, _vp, _i64, _vp]),
    "arcq_gemm_route": (ctypes.c_int, [_i64, _i64, _i64, ctypes.POINTER(Route)]),
    "arcq_mx_gemm_route": (ctypes.c_int, [_i64, _i64, _i64, ctypes.c_int, ctypes.POINTER(Route)]),
    "arcq_gemm_rest": (ctypes.c_int, [_i64, _i64, _i64, ctypes.POINTER(Rest)]),
    "arcq_mx_gemm_rest": (ctypes.c_int, [_i64, _i64, _i64, ctypes.c_int, ctypes.POINTER(Rest)]),
    "arcq_gemm_stream_tiles": (ctypes.c_int, [_i64, _i64, _i64, ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]),
    "arcq_mx_gemm_stream_tiles": (ctypes.c_int, [_i64, _i64, _i64, ctypes.c_int, ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]),
    "arcq_tile_order": (ctypes.c_int, [_i64, _i64, _vp, _vp]),
    "arcq_check_perm": (ctypes.c_int, [_vp, _i64, _vp, ctypes.POINTER(ctypes.c_int), _vp]),
}


class ArcqError(RuntimeError):
    def __init__(self, status, message):
        super().__init__(f"libarcq status {status}: {message}")
        self.status = status


_lib = None


def lib():
    """The loaded library; raises if it has not been built (no fallback exists)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: run `python -m paper_2601_07475_amd.build`")
        handle = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in SIGNATURES.items():
            fn = getattr(handle, name)
            fn.restype, fn.argtypes = res, args
        _lib = handle
    return _lib


def _check(status):
    if status != OK:
        raise ArcqError(status, lib().arcq_last_error().decode())


def _stream():
    """Handle of the current device's current stream.  torch.cuda.current_stream() builds a Stream object to tell it, 2.7 us of the 11
    that a call took on the host; the functions below it are private to torch, so another torch may not have them."""
    try:
        return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
    except AttributeError:
        return torch.cuda.current_stream().cuda_stream


def _ptr(t):
    """Address of a tensor's data; empty tensors and None are null.  (Every pointer argument is declared void*: plain integers do.)"""
    return t.data_ptr() or None if t is not None and t.numel() else None


def arcq_version():
    return lib().arcq_version()


def arcq_packed_sizes(rows, K, S):
    c, s = _sz(0), _sz(0)
    _check(lib().arcq_packed_sizes(rows, K, S, ctypes.byref(c), ctypes.byref(s)))
    return c.value, s.value


def _rows(x, perm):
    """(rows, K, pitch) of the input of a quantizer, checked."""
    assert x.is_cuda and x.dtype is torch.float16 and x.dim() == 2
    assert perm.is_cuda and perm.dtype is torch.int32 and perm.is_contiguous()
    rows, K = x.shape
    pitch, step = x.stride()
    assert step == 1
    if perm.numel() != K:
        raise ArcqError(BAD_SHAPE, "perm must have K entries")
    return rows, K, pitch if rows > 1 else max(K, pitch)


def _outputs(x, rows, code_bytes, scale_bytes, code_row, scale_row, codes, scales):
    """The output tensors of a quantizer: the caller's, checked, or new ones."""
    if codes is None:
        codes = x.new_empty((rows, code_row), dtype=torch.uint8)
    if scales is None:
        scales = x.new_empty((rows, scale_row), dtype=torch.uint8)
    assert codes.numel() == code_bytes and scales.numel() == scale_bytes and codes.is_contiguous() and scales.is_contiguous()
    return codes, scales


def _quantize(fn, x, perm, S, tensor_scale, codes=None, scales=None):
    rows, K, ldx = _rows(x, perm)
    cb, sb = arcq_packed_sizes(rows, K, S)
    codes, scales = _outputs(x, rows, cb, sb, (K + S) // 2, (K + S) // 16, codes, scales)
    _check(fn(_ptr(x), rows, K, ldx, _ptr(perm), S, float(tensor_scale), _ptr(codes), _ptr(scales), _stream()))
    return codes, scales


def arcq_quantize_act(x, perm, S, tensor_scale, codes=None, scales=None):
    """x fp16 [M, K] cuda, perm int32 [K] cuda -> (codes uint8 [M, K'/2], scales uint8 [M, K'/16])."""
    return _quantize(lib().arcq_quantize_act, x, perm, S, tensor_scale, codes, scales)


def arcq_rmsnorm_quantize_act(x, gamma, eps, perm, S, tensor_scale, codes=None, scales=None):
    """RMSNorm (weight gamma fp16 [K], eps) fused in front of arcq_quantize_act."""
    assert gamma.is_cuda and gamma.dtype == torch.float16 and gamma.is_contiguous() and gamma.numel() == x.shape[1]
    lib_fn = lib().arcq_rmsnorm_quantize_act

    def fn(xp, rows, K, ldx, permp, S_, sT, cp, sp, st):
        return lib_fn(xp, rows, K, ldx, _ptr(gamma), float(eps), permp, S_, sT, cp, sp, st)
    return _quantize(fn, x, perm, S, tensor_scale, codes, scales)


def arcq_pack_weight(w, perm, S, tensor_scale, codes=None, scales=None):
    """w fp16 [N, K] cuda -> packed [N, K'] with the outlier blocks duplicated."""
    return _quantize(lib().arcq_pack_weight, w, perm, S, tensor_scale, codes, scales)


def _with_flags(lib_fn, flags):
    """The *_ex entry points take `flags` right before the output pointers."""
    def fn(xp, rows, K, ldx, permp, S_, sT, cp, sp, st):
        return lib_fn(xp, rows, K, ldx, permp, S_, sT, int(flags), cp, sp, st)
    return fn


def arcq_quantize_act_ex(x, perm, S, tensor_scale, flags, codes=None, scales=None):
    """arcq_quantize_act with the layout / scale-rounding variants (LAYOUT_INTERLEAVED | SCALE_ROUND_UP)."""
    return _quantize(_with_flags(lib().arcq_quantize_act_ex, flags), x, perm, S, tensor_scale, codes, scales)


def arcq_rmsnorm_quantize_act_ex(x, gamma, eps, perm, S, tensor_scale, flags, codes=None, scales=None):
    assert gamma.is_cuda and gamma.dtype == torch.float16 and gamma.is_contiguous() and gamma.numel() == x.shape[1]
    lib_fn = lib().arcq_rmsnorm_quantize_act_ex

    def fn(xp, rows, K, ldx, permp, S_, sT, cp, sp, st):
        return lib_fn(xp, rows, K, ldx, _ptr(gamma), float(eps), permp, S_, sT, int(flags), cp, sp, st)
    return _quantize(fn, x, perm, S, tensor_scale, codes, scales)


def arcq_pack_weight_ex(w, perm, S, tensor_scale, flags, codes=None, scales=None):
    return _quantize(_with_flags(lib().arcq_pack_weight_ex, flags), w, perm, S, tensor_scale, codes, scales)


def arcq_gemm_workspace_size(M, N, Kp):
    b = _sz(0)
    _check(lib().arcq_gemm_workspace_size(M, N, Kp, ctypes.byref(b)))
    return b.value


def _operands(a_codes, a_scales, w_codes, w_scales, block):
    """(M, N, K') of packed operands, checked."""
    for t in (a_codes, a_scales, w_codes, w_scales):
        assert t.is_cuda and t.dtype is torch.uint8 and t.is_contiguous()
    a_shape, w_shape = a_codes.shape, w_codes.shape
    M, N, half = a_shape[0], w_shape[0], a_shape[1]
    if w_shape[1] != half or a_scales.shape != (M, 2 * half // block) or w_scales.shape != (N, 2 * half // block):
        raise ArcqError(BAD_SHAPE, "operand shapes disagree on K'")
    return M, N, 2 * half


def arcq_gemm(a_codes, a_scales, a_tensor_scale, w_codes, w_scales, w_tensor_scale,
              out_dtype=torch.float16, y=None, workspace=None):
    """y[M, N] = deq(A) deq(W)^T over K' (fp32 accumulate); returns y."""
    M, N, Kp = _operands(a_codes, a_scales, w_codes, w_scales, 16)
    if y is None:
        y = a_codes.new_empty((M, N), dtype=out_dtype)
    assert y.shape == (M, N) and y.stride(1) == 1 and y.dtype in (torch.float16, torch.float32)
    need = arcq_gemm_workspace_size(M, N, Kp)
    if need and (workspace is None or workspace.numel() * workspace.element_size() < need):
        workspace = torch.empty(need, dtype=torch.uint8, device=a_codes.device)
    ws_bytes = workspace.numel() * workspace.element_size() if workspace is not None else 0
    ldy = y.stride(0) if M > 1 else max(N, y.stride(0))
    _check(lib().arcq_gemm(_ptr(a_codes), _ptr(a_scales), float(a_tensor_scale),
                           _ptr(w_codes), _ptr(w_scales), float(w_tensor_scale), M, N, Kp,
                           _ptr(y), DTYPE_F16 if y.dtype == torch.float16 else DTYPE_F32, ldy,
                           _ptr(workspace), ws_bytes, _stream()))
    return y


NOALLOC_SCRATCH_BYTES = 8 << 20


def arcq_gemm_noalloc(a_codes, a_scales, a_tensor_scale, w_codes, w_scales, w_tensor_scale, y):
    """arcq_gemm without a workspace argument: split-K partial results go to the library's built-in scratch.
    The output tensor y [M, N] (fp16 or fp32) is the caller's; nothing is allocated here or in the library."""
    M, N, Kp = _operands(a_codes, a_scales, w_codes, w_scales, 16)
    assert y.shape == (M, N) and y.stride(1) == 1 and y.dtype in (torch.float16, torch.float32)
    ldy = y.stride(0) if M > 1 else max(N, y.stride(0))
    _check(lib().arcq_gemm_noalloc(_ptr(a_codes), _ptr(a_scales), float(a_tensor_scale),
                                   _ptr(w_codes), _ptr(w_scales), float(w_tensor_scale), M, N, Kp,
                                   _ptr(y), DTYPE_F16 if y.dtype == torch.float16 else DTYPE_F32, ldy, _stream()))
    return y


def arcq_calib_absmax(x, colmax):
    """Folds x fp16 [M, K] into the running per-channel abs-max colmax fp32 [K] (zeros before the first batch)."""
    assert x.is_cuda and x.dtype == torch.float16 and x.dim() == 2 and x.stride(1) == 1
    assert colmax.is_cuda and colmax.dtype == torch.float32 and colmax.is_contiguous() and colmax.numel() == x.shape[1]
    M, K = x.shape
    _check(lib().arcq_calib_absmax(_ptr(x), M, K, x.stride(0) if M > 1 else max(K, x.stride(0)), _ptr(colmax), _stream()))
    return colmax


def arcq_calib_select(colmax, perm=None, info=None):
    """colmax fp32 [K] -> (perm int32 [K], S, info int32 [4] = {S, S_raw, bits(max), bits(tau)}); synchronises."""
    assert colmax.is_cuda and colmax.dtype == torch.float32 and colmax.is_contiguous()
    K = colmax.numel()
    if perm is None:
        perm = torch.empty(K, dtype=torch.int32, device=colmax.device)
    if info is None:
        info = torch.empty(4, dtype=torch.int32, device=colmax.device)
    # page-locked: the kernel writes S itself (device named: torch's default one may be another)
    S = torch.empty(1, dtype=torch.int32, device="cpu", pin_memory=True)
    _check(lib().arcq_calib_select(_ptr(colmax), K, _ptr(perm), _ptr(info), _ptr(S), _stream()))
    return perm, S.item(), info


def _mx_quantize(fn, x, perm, S, codes=None, scales=None):
    rows, K, ldx = _rows(x, perm)
    cb, sb = _sz(0), _sz(0)
    _check(lib().arcq_mx_packed_sizes(rows, K, S, ctypes.byref(cb), ctypes.byref(sb)))
    codes, scales = _outputs(x, rows, cb.value, sb.value, (K + S) // 2, (K + S) // 32, codes, scales)
    _check(fn(_ptr(x), rows, K, ldx, _ptr(perm), S, _ptr(codes), _ptr(scales), _stream()))
    return codes, scales


def arcq_mx_quantize_act(x, perm, S, codes=None, scales=None):
    """MXFP4: x fp16 [M, K] -> (codes uint8 [M, K'/2], scales uint8 [M, K'/32])."""
    return _mx_quantize(lib().arcq_mx_quantize_act, x, perm, S, codes, scales)


def arcq_mx_pack_weight(w, perm, S, codes=None, scales=None):
    return _mx_quantize(lib().arcq_mx_pack_weight, w, perm, S, codes, scales)


def _mx_with_flags(lib_fn, flags):
    def fn(xp, rows, K, ldx, permp, S_, cp, sp, st):
        return lib_fn(xp, rows, K, ldx, permp, S_, int(flags), cp, sp, st)
    return fn


def arcq_mx_quantize_act_ex(x, perm, S, flags, codes=None, scales=None):
    return _mx_quantize(_mx_with_flags(lib().arcq_mx_quantize_act_ex, flags), x, perm, S, codes, scales)


def arcq_mx_pack_weight_ex(w, perm, S, flags, codes=None, scales=None):
    return _mx_quantize(_mx_with_flags(lib().arcq_mx_pack_weight_ex, flags), w, perm, S, codes, scales)


def arcq_mx_gemm_workspace_size(M, N, Kp):
    b = _sz(0)
    _check(lib().arcq_mx_gemm_workspace_size(M, N, Kp, ctypes.byref(b)))
    return b.value


def arcq_mx_gemm(a_codes, a_scales, w_codes, w_scales, out_dtype=torch.float16, y=None, workspace=None):
    """MXFP4: y[M, N] = deq(A) deq(W)^T over K' on the scaled FP4 matrix instruction; returns y.
    workspace: a uint8 tensor of at least arcq_mx_gemm_workspace_size bytes lets few-tile problems split K'
    (arcq_mx_gemm_ws); without one the plain entry point runs."""
    M, N, Kp = _operands(a_codes, a_scales, w_codes, w_scales, 32)
    if y is None:
        y = a_codes.new_empty((M, N), dtype=out_dtype)
    assert y.shape == (M, N) and y.stride(1) == 1 and y.dtype in (torch.float16, torch.float32)
    ldy = y.stride(0) if M > 1 else max(N, y.stride(0))
    dt = DTYPE_F16 if y.dtype == torch.float16 else DTYPE_F32
    if workspace is not None:
        assert workspace.is_cuda and workspace.is_contiguous()
        _check(lib().arcq_mx_gemm_ws(_ptr(a_codes), _ptr(a_scales), _ptr(w_codes), _ptr(w_scales), M, N, Kp, _ptr(y), dt, ldy,
                                     _ptr(workspace), workspace.numel() * workspace.element_size(), _stream()))
    else:
        _check(lib().arcq_mx_gemm(_ptr(a_codes), _ptr(a_scales), _ptr(w_codes), _ptr(w_scales), M, N, Kp, _ptr(y), dt, ldy,
                                  _stream()))
    return y


def _prepared(fn, args):
    """fn(*args) as a zero-argument callable.  The arguments are converted to their C types here, once: converting them on every
    call took 1.4 of its 3.1 us."""
    bound = tuple(None if a is None else ctype(a) for ctype, a in zip(fn.argtypes, args))

    def call():
        status = fn(*bound)
        if status != OK:
            _check(status)
    return call


def prepare_quantize_act(x, perm, S, tensor_scale, codes, scales):
    """Marshals the arguments of arcq_quantize_act once; returns a zero-argument callable that
    enqueues the call on the stream that was current at preparation time (for tight loops)."""
    rows, K = x.shape
    fn = lib().arcq_quantize_act
    args = (_ptr(x), rows, K, x.stride(0) if rows > 1 else K, _ptr(perm), S, float(tensor_scale),
            _ptr(codes), _ptr(scales), _stream())
    return _prepared(fn, args)


def prepare_rmsnorm_quantize_act(x, gamma, eps, perm, S, tensor_scale, codes, scales):
    """Same for arcq_rmsnorm_quantize_act."""
    rows, K = x.shape
    fn = lib().arcq_rmsnorm_quantize_act
    args = (_ptr(x), rows, K, x.stride(0) if rows > 1 else K, _ptr(gamma), float(eps), _ptr(perm), S,
            float(tensor_scale), _ptr(codes), _ptr(scales), _stream())
    return _prepared(fn, args)


def prepare_gemm(a_codes, a_scales, a_tensor_scale, w_codes, w_scales, w_tensor_scale, y, workspace=None):
    """Same for arcq_gemm."""
    M, N, Kp = a_codes.shape[0], w_codes.shape[0], a_codes.shape[1] * 2
    need = arcq_gemm_workspace_size(M, N, Kp)
    ws_bytes = workspace.numel() * workspace.element_size() if workspace is not None else 0
    if need > ws_bytes:
        raise ArcqError(WORKSPACE_TOO_SMALL, f"workspace of {need} bytes needed")
    fn = lib().arcq_gemm
    args = (_ptr(a_codes), _ptr(a_scales), float(a_tensor_scale), _ptr(w_codes), _ptr(w_scales),
            float(w_tensor_scale), M, N, Kp, _ptr(y), DTYPE_F16 if y.dtype == torch.float16 else DTYPE_F32,
            y.stride(0) if M > 1 else N, _ptr(workspace) if workspace is not None else None, ws_bytes, _stream())
    return _prepared(fn, args)


def prepare_mx_quantize_act(x, perm, S, codes, scales):
    """Same for arcq_mx_quantize_act."""
    rows, K = x.shape
    fn = lib().arcq_mx_quantize_act
    args = (_ptr(x), rows, K, x.stride(0) if rows > 1 else K, _ptr(perm), S, _ptr(codes), _ptr(scales), _stream())
    return _prepared(fn, args)


def prepare_mx_gemm(a_codes, a_scales, w_codes, w_scales, y, workspace=None):
    """Same for arcq_mx_gemm (arcq_mx_gemm_ws when a workspace tensor is given)."""
    M, N, Kp = a_codes.shape[0], w_codes.shape[0], a_codes.shape[1] * 2
    head = (_ptr(a_codes), _ptr(a_scales), _ptr(w_codes), _ptr(w_scales), M, N, Kp, _ptr(y),
            DTYPE_F16 if y.dtype == torch.float16 else DTYPE_F32, y.stride(0) if M > 1 else N)
    if workspace is not None:
        fn = lib().arcq_mx_gemm_ws
        args = head + (_ptr(workspace), workspace.numel() * workspace.element_size(), _stream())
    else:
        fn = lib().arcq_mx_gemm
        args = head + (_stream(),)
    return _prepared(fn, args)


PROBE_SINK_FLOATS = 262144


def _probe(name, iters, sink):
    if sink is None:
        sink = torch.empty(PROBE_SINK_FLOATS, dtype=torch.float32, device="cuda")
    assert sink.is_cuda and sink.dtype == torch.float32 and sink.numel() >= PROBE_SINK_FLOATS and sink.is_contiguous()
    flop = ctypes.c_double(0.0)
    _check(getattr(lib(), name)(int(iters), _ptr(sink), ctypes.byref(flop), _stream()))
    return flop.value


def arcq_probe_mfma_f16(iters, sink=None):
    """Enqueues the fp16 matrix-rate probe; returns the floating-point operations of the launch."""
    return _probe("arcq_probe_mfma_f16", iters, sink)


def arcq_probe_mfma_fp4(iters, sink=None):
    """Enqueues the scaled-FP4 matrix-rate probe; returns the floating-point operations of the launch."""
    return _probe("arcq_probe_mfma_fp4", iters, sink)


PROBE_UNTOUCHED = 0xA5A5A5A5


def arcq_probe_buffer_copy(src, size, scalar, words):
    """The 256 words that one wave's copy of `words` words a lane leaves in LDS, from byte `scalar` of the first `size` bytes of src on."""
    assert src.is_cuda and src.is_contiguous() and src.numel() * src.element_size() >= max(size, scalar + 1024)
    out = torch.empty(256, dtype=torch.int32, device="cuda")
    _check(lib().arcq_probe_buffer_copy(_ptr(src), size, scalar, words, _ptr(out), _stream()))
    return out


def arcq_gemm_route(M, N, Kp):
    """(kernel, tile rows, tile columns, runs of K', ahead) arcq_gemm takes for these sizes; no GPU needed."""
    r = Route()
    _check(lib().arcq_gemm_route(M, N, Kp, ctypes.byref(r)))
    return r.kernel, r.tile_rows, r.tile_cols, r.runs, r.ahead


def arcq_gemm_rest(M, N, Kp):
    """(rows, columns, (kernel, tile rows, tile columns)) of arcq_gemm's second launch, the last of the output; None: there is none."""
    r = Rest()
    _check(lib().arcq_gemm_rest(M, N, Kp, ctypes.byref(r)))
    return (r.rows, r.cols, (r.route.kernel, r.route.tile_rows, r.route.tile_cols)) if r.rows else None


def arcq_tile_order(tiles_m, tiles_n):
    """(tile row, tile column) of every workgroup of a tiled GEMM; no GPU needed."""
    rows, cols = (torch.empty(tiles_m * tiles_n, dtype=torch.int32, device="cpu") for _ in range(2))
    _check(lib().arcq_tile_order(tiles_m, tiles_n, _ptr(rows), _ptr(cols)))
    return list(zip(rows.tolist(), cols.tolist()))


def arcq_mx_gemm_rest(M, N, Kp, with_workspace=False):
    """The same for arcq_mx_gemm, with or without a workspace."""
    r = Rest()
    _check(lib().arcq_mx_gemm_rest(M, N, Kp, int(with_workspace), ctypes.byref(r)))
    return (r.rows, r.cols, (r.route.kernel, r.route.tile_rows, r.route.tile_cols)) if r.rows else None


def arcq_mx_gemm_route(M, N, Kp, with_workspace=False):
    """The same for arcq_mx_gemm, with or without a workspace."""
    r = Route()
    _check(lib().arcq_mx_gemm_route(M, N, Kp, int(with_workspace), ctypes.byref(r)))
    return r.kernel, r.tile_rows, r.tile_cols, r.runs, r.ahead


def arcq_gemm_stream_tiles(M, N, Kp):
    """(weight tiles a wave takes, those of the waves behind the first 16384 weight rows) where arcq_gemm streams, else (0, 0); no GPU needed."""
    tiles, behind = ctypes.c_int32(), ctypes.c_int32()
    _check(lib().arcq_gemm_stream_tiles(M, N, Kp, ctypes.byref(tiles), ctypes.byref(behind)))
    return tiles.value, behind.value


def arcq_mx_gemm_stream_tiles(M, N, Kp, with_workspace=False):
    """The same for arcq_mx_gemm, with or without a workspace."""
    tiles, behind = ctypes.c_int32(), ctypes.c_int32()
    _check(lib().arcq_mx_gemm_stream_tiles(M, N, Kp, int(with_workspace), ctypes.byref(tiles), ctypes.byref(behind)))
    return tiles.value, behind.value


def arcq_check_perm(perm):
    """True if the int32 cuda tensor perm is a permutation of 0..K-1 (synchronises)."""
    K = perm.numel()
    flags = torch.empty(K, dtype=torch.uint8, device=perm.device)
    res = ctypes.c_int(-1)
    _check(lib().arcq_check_perm(_ptr(perm), K, _ptr(flags), ctypes.byref(res), _stream()))
    return res.value == 1


def prepare_ref_gemm_bf16(x, w, y):
    """The hand-written bf16 comparison GEMM y = x w^T (x [M, K], w [N, K] bf16, y [M, N] fp16) as a prepared call."""
    for t in (x, w):
        assert t.is_cuda and t.dtype == torch.bfloat16 and t.is_contiguous()
    M, K = x.shape
    N = w.shape[0]
    assert w.shape[1] == K and y.shape == (M, N) and y.dtype == torch.float16 and y.stride(1) == 1
    fn = lib().arcq_ref_gemm_bf16
    args = (_ptr(x), _ptr(w), M, N, K, _ptr(y), y.stride(0) if M > 1 else N, _stream())
    return _prepared(fn, args)


def arcq_ref_gemm_bf16(x, w, y=None):
    if y is None:
        y = torch.empty((x.shape[0], w.shape[0]), dtype=torch.float16, device=x.device)
    prepare_ref_gemm_bf16(x, w, y)()
    return y

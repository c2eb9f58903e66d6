"""Binding of libaweq.so: same names and argument order as include/aweq.h.

Argument marshalling only, by the extension module _native (host functions: ctypes).  Tensor arguments are torch tensors
living on the GPU (or None for a nullable pointer); their data_ptr() is handed to the library, and the current torch
stream is passed unless `stream` is given.  PyTorch is used for device memory and streams
only.  Raw integer addresses are accepted in place of tensors (used by host-side tests).
"""
import ctypes as C
import importlib.machinery
import importlib.util
import os

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libaweq.so")
_NATIVE_PATH = os.path.join(_HERE, "_native" + importlib.machinery.EXTENSION_SUFFIXES[0])   # (the suffix that names this interpreter)
_lib = None
_calls = None    # the extension module, bound to the library
_torch = None

AWEQ_F32, AWEQ_F16, AWEQ_I8 = 0, 1, 2
OP_CALIB_STATS, OP_EQUALIZE, OP_QUANT_WEIGHT, OP_W8A8_GEMM, OP_BIAS_CORRECT, OP_WONLY_GEMM, OP_QUANT_ACT, OP_CALIBRATE = range(8)
BIAS_W8A8, BIAS_WEIGHT_ONLY = 0, 1
SCALE_NONE, SCALE_RANGE, SCALE_ABSMAX = 0, 1, 2
ST_DEGENERATE, ST_NONFINITE, ST_BIGQUOT, ST_SCALEGUARD, ST_ZEROPOINT = 1, 2, 4, 8, 16

EXPORTS = ("aweq_workspace_size", "aweq_status_string", "aweq_calib_stats", "aweq_equalize",
           "aweq_quant_weight", "aweq_quant_act", "aweq_w8a8_gemm", "aweq_bias_correct",
           "aweq_panel_bytes", "aweq_pack_panels_i8", "aweq_unpack_panels_i8", "aweq_wonly_gemm", "aweq_fold_quant_weight", "aweq_w8a8_gemm_fused",
           "aweq_calib_stats_static", "aweq_calibrate")
STATIC_SCRATCH_BYTES = 16 << 20

_vp, _i64, _i32, _u64, _f32, _sz = C.c_void_p, C.c_int64, C.c_int, C.c_uint64, C.c_float, C.c_size_t


class AweqError(RuntimeError):
    def __init__(self, code, name):
        super().__init__(f"libaweq: {name} ({code})")
        self.code = code
        self.name = name


def load_library():
    """Load the in-tree libaweq.so; raises if it has not been built (no fallback)."""
    global _lib, _calls, _torch
    if _lib is not None:
        return _lib
    # torch brings its own HIP runtime; it has to be the one already in the process when
    # libaweq.so resolves its runtime symbols, or streams and kernels end up in two runtimes
    import torch
    for path in (_LIB_PATH, _NATIVE_PATH):
        if not os.path.exists(path):
            raise ImportError(f"{path} is missing: build it with `python -m paper_2311_01305_amd.build` "
                              "(there is no CPU fallback)")
    lib = C.CDLL(_LIB_PATH)
    lib.aweq_workspace_size.restype = _sz
    lib.aweq_workspace_size.argtypes = [_i32, _i64, _i64, _i64]
    lib.aweq_status_string.restype = C.c_char_p
    lib.aweq_status_string.argtypes = [_i32]
    lib.aweq_panel_bytes.restype = _sz
    lib.aweq_panel_bytes.argtypes = [_i64, _i64]
    lib.aweq_pack_panels_i8.restype = _i32
    lib.aweq_pack_panels_i8.argtypes = [_vp, _i64, _i64, _i64, _vp, _vp]
    lib.aweq_unpack_panels_i8.restype = _i32
    lib.aweq_unpack_panels_i8.argtypes = [_vp, _i64, _i64, _vp, _i64, _vp]
    spec = importlib.util.spec_from_loader("_native", importlib.machinery.ExtensionFileLoader("_native", _NATIVE_PATH))
    calls = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(calls)
    for name in dir(calls):
        if name.startswith("aweq_"):
            calls.bind(name, C.cast(getattr(lib, name), C.c_void_p).value)
    _torch, _calls = torch, calls
    _lib = lib
    return lib


def _native():
    load_library()
    return _calls


def _ptr(t):
    if t is None:
        return None
    if isinstance(t, int):
        return t
    return t.data_ptr()


def _nbytes(t):
    return 0 if t is None else t.nbytes


def _stream(stream):
    if stream is not None:
        return stream if isinstance(stream, int) else stream.cuda_stream
    # the raw handle of the current device's current stream: torch.cuda.current_stream() builds a Stream object around it,
    # which took 3.9 us of a call that takes 5.6 without it (one decoded token, weight-only; 0.3 us this way)
    t = _torch
    if t is None:
        load_library()
        t = _torch
    if t.cuda.is_initialized():
        return t._C._cuda_getCurrentRawStream(t._C._cuda_getDevice())
    return t.cuda.current_stream().cuda_stream if t.cuda.is_available() else None


def _check(code):
    if code != 0:
        raise AweqError(code, aweq_status_string(code))


def aweq_status_string(code):
    return load_library().aweq_status_string(int(code)).decode()


def aweq_workspace_size(op, rows, K, N=0):
    return int(load_library().aweq_workspace_size(int(op), int(rows), int(K), int(N)))


def aweq_calib_stats(M, dt, rows, K, ld, cmin, cmax, csum, count, accumulate, finalize, r, R, p, ws,
                     status=None, stream=None, ws_bytes=None):
    _check((_calls or _native()).aweq_calib_stats(
        M, dt, rows, K, ld, cmin, cmax, csum, count, int(accumulate), int(finalize),
        r, R, p, ws, _nbytes(ws) if ws_bytes is None else ws_bytes, status,
        _stream(stream)))


def aweq_calib_stats_static(M, dt, rows, K, ld, cmin, cmax, csum, count, accumulate, finalize, r, R, p,
                            status=None, stream=None):
    _check((_calls or _native()).aweq_calib_stats_static(
        M, dt, rows, K, ld, cmin, cmax, csum, count, int(accumulate), int(finalize),
        r, R, p, status, _stream(stream)))


def aweq_equalize(xmin, xmax, xsum, count, wmin, wmax, K, enable_awe, s, inv_s, W, W_hat, dt, N, ldw, ldwh,
                  prev_scale, xhat_range, mu_xhat, act_step, act_zero, status=None, stream=None):
    _check((_calls or _native()).aweq_equalize(
        xmin, xmax, xsum, int(count), wmin, wmax, K, int(enable_awe), s,
        inv_s, W, W_hat, dt, N, ldw, ldwh, prev_scale, xhat_range, mu_xhat,
        act_step, act_zero, status, _stream(stream)))


def aweq_quant_weight(W_hat, dt, N, K, ldw, bits, group, codes, step, zero, rowsum_w, ws=None,
                      status=None, stream=None, ws_bytes=None):
    _check((_calls or _native()).aweq_quant_weight(
        W_hat, dt, N, K, ldw, int(bits), int(group), codes, step, zero, rowsum_w,
        ws, _nbytes(ws) if ws_bytes is None else ws_bytes, status, _stream(stream)))


def aweq_quant_act(X, dt, T, K, ldx, inv_s, act_step, act_zero, xq, rowsum_x, colsum_xq, ws=None, status=None, stream=None,
                   ws_bytes=None):
    _check((_calls or _native()).aweq_quant_act(
        X, dt, T, K, ldx, inv_s, act_step, act_zero, xq, rowsum_x,
        colsum_xq, ws, _nbytes(ws) if ws_bytes is None else ws_bytes, status, _stream(stream)))


def aweq_w8a8_gemm(X, x_dt, T, K, ldx, inv_s, act_step, act_zero, xq, rowsum_x, colsum_xq, wq, N, step_w, zero_w, w_group,
                   rowsum_w, bias, out_i32, out_deq, out_dt, ldo, colsum_acc, ws=None, status=None, stream=None,
                   ws_bytes=None):
    _check((_calls or _native()).aweq_w8a8_gemm(
        X, x_dt, T, K, ldx, inv_s, act_step, act_zero, xq, rowsum_x,
        colsum_xq, wq, N, step_w, zero_w, int(w_group), rowsum_w, bias, out_i32,
        out_deq, out_dt, ldo, colsum_acc, ws, _nbytes(ws) if ws_bytes is None else ws_bytes,
        status, _stream(stream)))


def aweq_bias_correct(mode, W_hat, dt, N, K, ldw, mu_xhat, count, colsum_acc, colsum_xq, rowsum_w, act_step,
                      act_zero, codes, bits, group, step_w, zero_w, bias_in, delta, bias_out, enable_bc,
                      status=None, stream=None):
    _check((_calls or _native()).aweq_bias_correct(
        int(mode), W_hat, dt, N, K, ldw, mu_xhat, int(count), colsum_acc, colsum_xq,
        rowsum_w, act_step, act_zero, codes, int(bits), int(group), step_w,
        zero_w, bias_in, delta, bias_out, int(enable_bc), status, _stream(stream)))


def aweq_panel_bytes(rows, K):
    return int(load_library().aweq_panel_bytes(int(rows), int(K)))


def aweq_pack_panels_i8(src, rows, K, ld, panels, stream=None):
    _check(load_library().aweq_pack_panels_i8(_ptr(src), rows, K, ld, _ptr(panels), _stream(stream)))


def aweq_unpack_panels_i8(panels, rows, K, dst, ld, stream=None):
    _check(load_library().aweq_unpack_panels_i8(_ptr(panels), rows, K, _ptr(dst), ld, _stream(stream)))


def aweq_w8a8_gemm_fused(xq, T, K, wq, N, act_step, act_zero, step_w, zero_w, rowsum_x, rowsum_w, bias, act, out_f16, ldo,
                         colsum_acc, ycmin=None, ycmax=None, ycsum=None, ycount=None, accumulate=0, next_inv_s=None,
                         next_step=None, next_zero=None, yq=None, rowsum_y=None, colsum_yq=None, ws=None, status=None,
                         stream=None, ws_bytes=None):
    _check((_calls or _native()).aweq_w8a8_gemm_fused(
        xq, T, K, wq, N, act_step, act_zero, step_w, zero_w, rowsum_x,
        rowsum_w, bias, int(act), out_f16, ldo, colsum_acc, ycmin, ycmax, ycsum,
        ycount, int(accumulate), next_inv_s, next_step, next_zero, yq, rowsum_y,
        colsum_yq, ws, (_nbytes(ws) if ws is not None else 0) if ws_bytes is None else ws_bytes, status,
        _stream(stream)))


def aweq_wonly_gemm(X_hat, T, K, ldx, codes, bits, group, step_w, zero_w, N, bias, out, out_dt, ldo, ws,
                    status=None, stream=None, ws_bytes=None):
    _check((_calls or _native()).aweq_wonly_gemm(X_hat, T, K, ldx, codes, int(bits), int(group), step_w,
                                          zero_w, N, bias, out, out_dt, ldo, ws,
                                          _nbytes(ws) if ws_bytes is None else ws_bytes, status,
                                          _stream(stream)))


def aweq_fold_quant_weight(W, dt, N, K, ldw, s, W_hat, ldwh, bits, codes, step, zero, rowsum_w, status=None, stream=None):
    _check((_calls or _native()).aweq_fold_quant_weight(W, dt, N, K, ldw, s, W_hat, ldwh, int(bits), codes,
                                                 step, zero, rowsum_w, status, _stream(stream)))


def aweq_calibrate(layer, weights, stream=None):
    """layer: the fields of aweq_calib_layer in order; weights: a sequence of the fields of aweq_calib_weight in order.  Tensors, addresses,
    integers or None."""
    _check((_calls or _native()).aweq_calibrate(layer, weights, _stream(stream)))

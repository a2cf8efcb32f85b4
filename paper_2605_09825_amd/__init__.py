"""Python binding of libmxfp4.so (the gfx950 MXFP4 linear-layer library).

Argument marshalling only: every function here forwards to the C-ABI entry point
of the same name (include/mxfp4.h) with raw device pointers and the current torch
stream; torch is used for device memory and streams and for nothing else.  There is
no fallback: if the HIP library is missing or a call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Tuple

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libmxfp4.so")
if os.environ.get("MXFP4_SANITIZE_HOST", "") not in ("", "0"):  # host-sanitizer build (see build.py)
    LIB_PATH = os.path.join(HERE, "libmxfp4_san.so")

# enums of include/mxfp4.h
OK, EINVAL, ESHAPE, EALIGN, EWORKSPACE, EDEVICE, ENOTIMPL = range(7)
AXIS_LAST, AXIS_FIRST = 0, 1
HAD_NONE, HAD_DET, HAD_RANDSIGN, HAD_DET16, HAD_RANDSIGN16 = 0, 1, 2, 3, 4
RNE, SR = 0, 1
OUT_BF16, OUT_FP32 = 0, 1
GEOM_1D, GEOM_2D = 0, 1
FMT_E2M1, FMT_E4M3 = 0, 1

EXPORTS = ("mxfp4_quantize", "mxfp4_quantize_dual", "mxfp4_quantize_2d", "mxfp4_quantize_fp8",
           "mxfp4_quantize_fp8_dual", "mxfp4_gemm",
           "mxfp4_gemm_fmt", "mxfp4_gemm_pair", "mxfp4_gemm_plan", "mxfp4_gemm_route",
           "mxfp4_gemm_pair_route", "mxfp4_linear_fwd", "mxfp4_linear_fwd_static", "mxfp4_linear_bwd",
           "mxfp4_linear_fwd_save", "mxfp4_linear_bwd_saved", "mxfp4_linear_saved_bytes",
           "mxfp4_linear_saved_layout", "mxfp4_linear_workspace_bytes", "mxfp4_linear_workspace_layout",
           "mxfp4_status_string")


class LinearCfg(ctypes.Structure):
    """mxfp4_linear_cfg"""
    _fields_ = [("hadamard", ctypes.c_int32), ("rounding", ctypes.c_int32), ("seed", ctypes.c_uint64),
                ("y_dtype", ctypes.c_int32), ("dx_dtype", ctypes.c_int32), ("dw_dtype", ctypes.c_int32),
                ("dw_accumulate", ctypes.c_int32), ("geometry", ctypes.c_int32), ("fprop_format", ctypes.c_int32),
                ("dgrad_format", ctypes.c_int32), ("wgrad_format", ctypes.c_int32)]


class Mxfp4Error(RuntimeError):
    def __init__(self, call: str, status: int):
        self.status = status
        super().__init__(f"{call} failed: status {status} ({status_string(status)})")


_lib: Optional[ctypes.CDLL] = None


def lib() -> ctypes.CDLL:
    """Load libmxfp4.so (built by paper_2605_09825_amd.build); raises if it is not there."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with "
                               "`python -m paper_2605_09825_amd.build` (there is no CPU fallback)")
        L = ctypes.CDLL(LIB_PATH)
        vp, i64, ci, u64, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_uint64, ctypes.c_size_t
        L.mxfp4_quantize.restype = ci
        L.mxfp4_quantize.argtypes = [vp, i64, i64, i64, ci, ci, ci, u64, vp, vp, vp]
        L.mxfp4_quantize_dual.restype = ci
        L.mxfp4_quantize_dual.argtypes = [vp, i64, i64, i64, ci, ci, u64, vp, vp, vp, vp, vp]
        L.mxfp4_quantize_fp8.restype = ci
        L.mxfp4_quantize_fp8.argtypes = [vp, i64, i64, i64, ci, ci, u64, vp, vp, vp]
        L.mxfp4_quantize_fp8_dual.restype = ci
        L.mxfp4_quantize_fp8_dual.argtypes = [vp, i64, i64, i64, ci, u64, vp, vp, vp, vp, vp]
        L.mxfp4_gemm_fmt.restype = ci
        L.mxfp4_gemm_fmt.argtypes = [vp, vp, ci, vp, vp, ci, i64, i64, i64, vp, i64, ci, ci, vp]
        L.mxfp4_quantize_2d.restype = ci
        L.mxfp4_quantize_2d.argtypes = [vp, i64, i64, i64, ci, ci, u64, vp, vp, vp, vp, vp]
        L.mxfp4_linear_fwd_save.restype = ci
        L.mxfp4_linear_fwd_save.argtypes = [vp, vp, vp, i64, i64, i64, ctypes.POINTER(LinearCfg), vp, sz, vp, sz, vp]
        L.mxfp4_linear_bwd_saved.restype = ci
        L.mxfp4_linear_bwd_saved.argtypes = [vp, vp, sz, vp, vp, i64, i64, i64, ctypes.POINTER(LinearCfg), vp, sz, vp]
        L.mxfp4_linear_saved_bytes.restype = sz
        L.mxfp4_linear_saved_bytes.argtypes = [i64, i64, i64, ctypes.POINTER(LinearCfg)]
        L.mxfp4_linear_saved_layout.restype = ci
        L.mxfp4_linear_saved_layout.argtypes = [i64, i64, i64, ctypes.POINTER(LinearCfg), ctypes.POINTER(sz)]
        L.mxfp4_gemm.restype = ci
        L.mxfp4_gemm.argtypes = [vp, vp, vp, vp, i64, i64, i64, vp, i64, ci, ci, vp]
        L.mxfp4_linear_fwd.restype = ci
        L.mxfp4_linear_fwd.argtypes = [vp, vp, vp, i64, i64, i64, ctypes.POINTER(LinearCfg), vp, sz, vp]
        L.mxfp4_gemm_pair.restype = ci
        L.mxfp4_gemm_pair.argtypes = ([vp, vp, vp, vp, i64, i64, i64, vp, i64, ci] +
                                      [vp, vp, vp, vp, i64, i64, i64, vp, i64, ci, ci] + [vp])
        L.mxfp4_gemm_plan.restype = ci
        L.mxfp4_gemm_plan.argtypes = [i64, i64, i64, ci, ci, i64, ci, ctypes.POINTER(ci), ctypes.POINTER(i64)]
        L.mxfp4_gemm_route.restype = ci
        L.mxfp4_gemm_route.argtypes = [i64, i64, i64, ci, ci, i64, ci, ci, ci, ctypes.POINTER(ci)]
        L.mxfp4_gemm_pair_route.restype = ci
        L.mxfp4_gemm_pair_route.argtypes = ([i64, i64, i64, ci, i64, ci] * 2) + [ci, ci, ctypes.POINTER(ci)]
        L.mxfp4_linear_fwd_static.restype = ci
        L.mxfp4_linear_fwd_static.argtypes = [vp, vp, vp, i64, i64, i64, ctypes.POINTER(LinearCfg), vp]
        L.mxfp4_linear_bwd.restype = ci
        L.mxfp4_linear_bwd.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, ctypes.POINTER(LinearCfg), vp, sz, vp]
        L.mxfp4_linear_workspace_bytes.restype = sz
        L.mxfp4_linear_workspace_bytes.argtypes = [i64, i64, i64, ctypes.POINTER(LinearCfg), ci]
        L.mxfp4_linear_workspace_layout.restype = ci
        L.mxfp4_linear_workspace_layout.argtypes = [i64, i64, i64, ctypes.POINTER(LinearCfg), ci, ctypes.POINTER(sz)]
        L.mxfp4_status_string.restype = ctypes.c_char_p
        L.mxfp4_status_string.argtypes = [ci]
        _lib = L
    return _lib


def status_string(status: int) -> str:
    return lib().mxfp4_status_string(int(status)).decode()


def _check(call: str, status: int) -> None:
    if status != OK:
        raise Mxfp4Error(call, status)


def _stream_ptr(stream) -> int:
    # (the handle of the current device's current stream, without the Stream object that torch.cuda.current_stream()
    # builds around it: 2.9 us of the 8 us that a call of a small product took on the host)
    if stream is not None:
        return int(stream.cuda_stream)
    import torch
    return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())


def _ptr(t) -> Optional[int]:
    return None if t is None else int(t.data_ptr())


def _out_dtype(code: int):
    import torch
    return torch.float32 if code == OUT_FP32 else torch.bfloat16


# ---------------------------------------------------------------------------------------
def mxfp4_quantize(x, axis: int = AXIS_LAST, hadamard: int = HAD_NONE, rounding: int = RNE, seed: int = 0,
                   q=None, s=None, stream=None) -> Tuple["torch.Tensor", "torch.Tensor"]:
    """x: bf16 CUDA tensor [rows][cols] with unit inner stride.  Returns (q, s) uint8 tensors
    [R][C/2] and [R][C/32] (allocated here with torch.empty unless passed in)."""
    import torch
    assert x.is_cuda and x.dtype == torch.bfloat16 and x.dim() == 2 and (x.numel() == 0 or x.stride(1) == 1)
    rows, cols = x.shape
    ld = x.stride(0) if rows > 1 else max(cols, x.stride(0))
    R, C = (rows, cols) if axis == AXIS_LAST else (cols, rows)
    if q is None:
        q = torch.empty((R, C // 2), dtype=torch.uint8, device=x.device)
    if s is None:
        s = torch.empty((R, C // 32), dtype=torch.uint8, device=x.device)
    _check("mxfp4_quantize", lib().mxfp4_quantize(_ptr(x), rows, cols, ld, axis, hadamard, rounding,
                                                  seed & (2**64 - 1), _ptr(q), _ptr(s), _stream_ptr(stream)))
    return q, s


def mxfp4_quantize_dual(x, hadamard: int = HAD_NONE, rounding: int = RNE, seed: int = 0, stream=None):
    """Both quantisations of x [rows][cols] from one pass: returns (q_last, s_last, q_first, s_first)."""
    import torch
    assert x.is_cuda and x.dtype == torch.bfloat16 and x.dim() == 2 and (x.numel() == 0 or x.stride(1) == 1)
    rows, cols = x.shape
    ld = x.stride(0) if rows > 1 else max(cols, x.stride(0))
    u8 = dict(dtype=torch.uint8, device=x.device)
    ql, sl = torch.empty((rows, cols // 2), **u8), torch.empty((rows, cols // 32), **u8)
    qf, sf = torch.empty((cols, rows // 2), **u8), torch.empty((cols, rows // 32), **u8)
    _check("mxfp4_quantize_dual", lib().mxfp4_quantize_dual(_ptr(x), rows, cols, ld, hadamard, rounding,
                                                            seed & (2**64 - 1), _ptr(ql), _ptr(sl), _ptr(qf),
                                                            _ptr(sf), _stream_ptr(stream)))
    return ql, sl, qf, sf


def mxfp4_quantize_2d(x, hadamard: int = HAD_NONE, rounding: int = RNE, seed: int = 0, want_last: bool = True,
                      want_first: bool = True, stream=None):
    """32 x 32 block scaling: returns (q_last, s_last, q_first, s_first); an output not wanted is None."""
    import torch
    assert x.is_cuda and x.dtype == torch.bfloat16 and x.dim() == 2 and (x.numel() == 0 or x.stride(1) == 1)
    rows, cols = x.shape
    ld = x.stride(0) if rows > 1 else max(cols, x.stride(0))
    u8 = dict(dtype=torch.uint8, device=x.device)
    ql = sl = qf = sf = None
    if want_last:
        ql, sl = torch.empty((rows, cols // 2), **u8), torch.empty((rows, cols // 32), **u8)
    if want_first:
        qf, sf = torch.empty((cols, rows // 2), **u8), torch.empty((cols, rows // 32), **u8)
    _check("mxfp4_quantize_2d", lib().mxfp4_quantize_2d(_ptr(x), rows, cols, ld, hadamard, rounding,
                                                        seed & (2**64 - 1), _ptr(ql), _ptr(sl), _ptr(qf), _ptr(sf),
                                                        _stream_ptr(stream)))
    return ql, sl, qf, sf


def mxfp4_quantize_fp8(x, axis: int = AXIS_LAST, hadamard: int = HAD_NONE, seed: int = 0, q=None, s=None,
                       stream=None):
    """MXFP8 (E4M3) quantisation of x [rows][cols]: returns (q8 [R][C], s [R][C/32])."""
    import torch
    assert x.is_cuda and x.dtype == torch.bfloat16 and x.dim() == 2 and (x.numel() == 0 or x.stride(1) == 1)
    rows, cols = x.shape
    ld = x.stride(0) if rows > 1 else max(cols, x.stride(0))
    R, C = (rows, cols) if axis == AXIS_LAST else (cols, rows)
    if q is None:
        q = torch.empty((R, C), dtype=torch.uint8, device=x.device)
    if s is None:
        s = torch.empty((R, C // 32), dtype=torch.uint8, device=x.device)
    _check("mxfp4_quantize_fp8", lib().mxfp4_quantize_fp8(_ptr(x), rows, cols, ld, axis, hadamard,
                                                          seed & (2**64 - 1), _ptr(q), _ptr(s), _stream_ptr(stream)))
    return q, s


def mxfp4_quantize_fp8_dual(x, hadamard: int = HAD_NONE, seed: int = 0, stream=None):
    """Both MXFP8 quantisations of x [rows][cols] from one pass: returns (q8_last, s_last, q8_first, s_first)."""
    import torch
    assert x.is_cuda and x.dtype == torch.bfloat16 and x.dim() == 2 and (x.numel() == 0 or x.stride(1) == 1)
    rows, cols = x.shape
    ld = x.stride(0) if rows > 1 else max(cols, x.stride(0))
    u8 = dict(dtype=torch.uint8, device=x.device)
    ql, sl = torch.empty((rows, cols), **u8), torch.empty((rows, cols // 32), **u8)
    qf, sf = torch.empty((cols, rows), **u8), torch.empty((cols, rows // 32), **u8)
    _check("mxfp4_quantize_fp8_dual", lib().mxfp4_quantize_fp8_dual(_ptr(x), rows, cols, ld, hadamard,
                                                                    seed & (2**64 - 1), _ptr(ql), _ptr(sl), _ptr(qf),
                                                                    _ptr(sf), _stream_ptr(stream)))
    return ql, sl, qf, sf


def mxfp4_gemm(a_q, a_s, b_q, b_s, out=None, out_dtype: int = OUT_FP32, accumulate: bool = False, stream=None,
               a_format: int = FMT_E2M1, b_format: int = FMT_E2M1):
    """out[i][j] (+)= sum_c A[i][c] B[j][c] on canonical quantised operands (uint8 CUDA tensors); with a format
    other than E2M1 for either operand the call goes to mxfp4_gemm_fmt."""
    import torch
    Ra, C = a_q.shape[0], a_q.shape[1] * (2 if a_format == FMT_E2M1 else 1)
    Rb = b_q.shape[0]
    assert b_q.shape[1] * (2 if b_format == FMT_E2M1 else 1) == C and a_q.is_contiguous() and b_q.is_contiguous()
    assert a_s.is_contiguous() and b_s.is_contiguous()
    if out is None:
        out = torch.empty((Ra, Rb), dtype=_out_dtype(out_dtype), device=a_q.device)
    assert out.dtype == _out_dtype(out_dtype) and (out.numel() == 0 or out.stride(1) == 1)
    ld = out.stride(0) if Ra > 1 else max(Rb, out.stride(0))
    if a_format == FMT_E2M1 and b_format == FMT_E2M1:
        _check("mxfp4_gemm", lib().mxfp4_gemm(_ptr(a_q), _ptr(a_s), _ptr(b_q), _ptr(b_s), Ra, Rb, C, _ptr(out), ld,
                                              out_dtype, int(accumulate), _stream_ptr(stream)))
    else:
        _check("mxfp4_gemm_fmt", lib().mxfp4_gemm_fmt(_ptr(a_q), _ptr(a_s), a_format, _ptr(b_q), _ptr(b_s), b_format,
                                                      Ra, Rb, C, _ptr(out), ld, out_dtype, int(accumulate),
                                                      _stream_ptr(stream)))
    return out


def mxfp4_gemm_pair(a0, b0, out0, a1, b1, out1, accumulate1: bool = False, stream=None):
    """Two independent MXFP4 GEMMs enqueued together (Dgrad and Wgrad of one layer): a0, b0, a1, b1 are
    (codes, scales) pairs of uint8 CUDA tensors, out0 / out1 preallocated bf16 or fp32 matrices."""
    import torch
    args = []
    for (aq, as_), (bq, bs), out in ((a0, b0, out0), (a1, b1, out1)):
        Ra, Rb, C = aq.shape[0], bq.shape[0], aq.shape[1] * 2
        assert bq.shape[1] * 2 == C and all(t.is_contiguous() for t in (aq, as_, bq, bs))
        assert tuple(out.shape) == (Ra, Rb) and (out.numel() == 0 or out.stride(1) == 1)
        ld = out.stride(0) if Ra > 1 else max(Rb, out.stride(0))
        args += [_ptr(aq), _ptr(as_), _ptr(bq), _ptr(bs), Ra, Rb, C, _ptr(out), ld,
                 OUT_FP32 if out.dtype == torch.float32 else OUT_BF16]
    _check("mxfp4_gemm_pair", lib().mxfp4_gemm_pair(*args, int(accumulate1), _stream_ptr(stream)))
    return out0, out1


GEMM_ANY, GEMM_TILED_256, GEMM_TILED_128, GEMM_TILED_256_TAIL_128 = 0, 1, 2, 3


def mxfp4_gemm_plan(Ra: int, Rb: int, C: int, a_format: int = FMT_E2M1, b_format: int = FMT_E2M1,
                    ld_out: Optional[int] = None, compute_units: int = 256):
    """The kernels a GEMM of this shape is cut into: list of (kind, r0, rows, c0, cols, main_tiles).  Host-only."""
    n = ctypes.c_int(0)
    parts = (ctypes.c_int64 * 24)()
    _check("mxfp4_gemm_plan", lib().mxfp4_gemm_plan(Ra, Rb, C, a_format, b_format, Rb if ld_out is None else ld_out,
                                                    compute_units, ctypes.byref(n), parts))
    return [tuple(int(parts[6 * i + k]) for k in range(6)) for i in range(n.value)]


ROUTE_NONE, ROUTE_BLOCKS, ROUTE_ANY_SHAPE, ROUTE_EDGE_64, ROUTE_EDGE_128, ROUTE_EDGE_256, ROUTE_RAGGED_TILED = range(-1, 6)
PAIR_APART, PAIR_SIDE_BY_SIDE, PAIR_NARROW_BESIDE_WIDE, PAIR_EDGE = range(4)


def mxfp4_gemm_route(Ra: int, Rb: int, C: int, a_format: int = FMT_E2M1, b_format: int = FMT_E2M1,
                     ld_out: Optional[int] = None, out_dtype: int = OUT_BF16, accumulate: bool = False,
                     compute_units: int = 256) -> int:
    """What mxfp4_gemm launches for a product of this shape (ROUTE_*).  Host-only."""
    route = ctypes.c_int(0)
    _check("mxfp4_gemm_route", lib().mxfp4_gemm_route(Ra, Rb, C, a_format, b_format, Rb if ld_out is None else ld_out,
                                                      out_dtype, int(accumulate), compute_units, ctypes.byref(route)))
    return route.value


def mxfp4_gemm_pair_route(shape0, shape1, formats=(FMT_E2M1, FMT_E2M1), out_dtypes=(OUT_BF16, OUT_FP32),
                          accumulate1: bool = False, compute_units: int = 256):
    """What mxfp4_gemm_pair, or a backward call with both gradients, launches for products of shapes (Ra, Rb, C) with
    dense outputs: (PAIR_*, first, n, cut).  Host-only."""
    route = (ctypes.c_int * 4)()
    (a0, b0, c0), (a1, b1, c1) = shape0, shape1
    _check("mxfp4_gemm_pair_route", lib().mxfp4_gemm_pair_route(
        a0, b0, c0, formats[0], b0, out_dtypes[0], a1, b1, c1, formats[1], b1, out_dtypes[1], int(accumulate1),
        compute_units, route))
    return tuple(int(v) for v in route)


def mxfp4_linear_workspace_bytes(M: int, N: int, K: int, cfg: LinearCfg, bwd: bool) -> int:
    return int(lib().mxfp4_linear_workspace_bytes(M, N, K, ctypes.byref(cfg), int(bwd)))


def _cfg_ref(cfg):
    return None if cfg is None else ctypes.byref(cfg)


def mxfp4_linear_workspace_layout(M: int, N: int, K: int, bwd: bool, cfg: Optional[LinearCfg] = None):
    arr = (ctypes.c_size_t * 8)()
    _check("mxfp4_linear_workspace_layout",
           lib().mxfp4_linear_workspace_layout(M, N, K, _cfg_ref(cfg), int(bwd), arr))
    return [int(v) for v in arr]


def make_cfg(hadamard: int = HAD_NONE, rounding: int = RNE, seed: int = 0, y_dtype: int = OUT_BF16,
             dx_dtype: int = OUT_BF16, dw_dtype: int = OUT_FP32, dw_accumulate: bool = False,
             geometry: int = GEOM_1D, fprop_format: int = FMT_E2M1, dgrad_format: int = FMT_E2M1,
             wgrad_format: int = FMT_E2M1) -> LinearCfg:
    return LinearCfg(hadamard, rounding, seed & (2**64 - 1), y_dtype, dx_dtype, dw_dtype, int(dw_accumulate),
                     geometry, fprop_format, dgrad_format, wgrad_format)


def mxfp4_linear_fwd(x, w, cfg: LinearCfg, y=None, workspace=None, stream=None):
    """Y = Q(X H) Q(W H)^T.  x [M][K], w [N][K] bf16 CUDA, contiguous.  Returns (y, workspace)."""
    import torch
    M, K = x.shape
    N = w.shape[0]
    assert w.shape[1] == K and x.is_contiguous() and w.is_contiguous()
    need = mxfp4_linear_workspace_bytes(M, N, K, cfg, False)
    if workspace is None:
        workspace = torch.empty(need, dtype=torch.uint8, device=x.device)
    if y is None:
        y = torch.empty((M, N), dtype=_out_dtype(cfg.y_dtype), device=x.device)
    _check("mxfp4_linear_fwd", lib().mxfp4_linear_fwd(_ptr(x), _ptr(w), _ptr(y), M, N, K, ctypes.byref(cfg),
                                                      _ptr(workspace), workspace.numel(), _stream_ptr(stream)))
    return y, workspace


STATIC_SCRATCH_BYTES = 32 << 20


def mxfp4_linear_fwd_static(x, w, cfg: LinearCfg, y, stream=None):
    """mxfp4_linear_fwd on the library's own static device scratch: no workspace, nothing allocated (y is the
    caller's).  Returns y."""
    M, K = x.shape
    N = w.shape[0]
    assert w.shape[1] == K and x.is_contiguous() and w.is_contiguous() and y.is_contiguous()
    _check("mxfp4_linear_fwd_static", lib().mxfp4_linear_fwd_static(_ptr(x), _ptr(w), _ptr(y), M, N, K,
                                                                    ctypes.byref(cfg), _stream_ptr(stream)))
    return y


def mxfp4_linear_bwd(dy, x, w, cfg: LinearCfg, dx=None, dw=None, need_dx: bool = True, need_dw: bool = True,
                     workspace=None, stream=None):
    """dX = Q(dY H) Q(W^T H)^T and dW = Q(dY^T H) Q(X^T H)^T.  Returns (dx, dw, workspace)."""
    import torch
    M, N = dy.shape
    K = x.shape[1] if x is not None else w.shape[1]
    need = mxfp4_linear_workspace_bytes(M, N, K, cfg, True)
    if workspace is None:
        workspace = torch.empty(need, dtype=torch.uint8, device=dy.device)
    if need_dx and dx is None:
        dx = torch.empty((M, K), dtype=_out_dtype(cfg.dx_dtype), device=dy.device)
    if need_dw and dw is None:
        assert not cfg.dw_accumulate, "accumulating into dW needs the caller's dW"
        dw = torch.empty((N, K), dtype=_out_dtype(cfg.dw_dtype), device=dy.device)
    _check("mxfp4_linear_bwd", lib().mxfp4_linear_bwd(_ptr(dy), _ptr(x), _ptr(w), _ptr(dx) if need_dx else None,
                                                      _ptr(dw) if need_dw else None, M, N, K, ctypes.byref(cfg),
                                                      _ptr(workspace), workspace.numel(), _stream_ptr(stream)))
    return dx, dw, workspace


def mxfp4_linear_saved_bytes(M: int, N: int, K: int, cfg: Optional[LinearCfg] = None) -> int:
    return int(lib().mxfp4_linear_saved_bytes(M, N, K, _cfg_ref(cfg)))


def mxfp4_linear_saved_layout(M: int, N: int, K: int, cfg: Optional[LinearCfg] = None):
    arr = (ctypes.c_size_t * 4)()
    _check("mxfp4_linear_saved_layout", lib().mxfp4_linear_saved_layout(M, N, K, _cfg_ref(cfg), arr))
    return [int(v) for v in arr]


def mxfp4_linear_fwd_save(x, w, cfg: LinearCfg, y=None, workspace=None, saved=None, stream=None):
    """mxfp4_linear_fwd that also leaves the column-wise quantisations of W and X in `saved` for
    mxfp4_linear_bwd_saved.  Returns (y, workspace, saved)."""
    import torch
    M, K = x.shape
    N = w.shape[0]
    assert w.shape[1] == K and x.is_contiguous() and w.is_contiguous()
    if workspace is None:
        workspace = torch.empty(mxfp4_linear_workspace_bytes(M, N, K, cfg, False), dtype=torch.uint8, device=x.device)
    if saved is None:
        saved = torch.empty(mxfp4_linear_saved_bytes(M, N, K, cfg), dtype=torch.uint8, device=x.device)
    if y is None:
        y = torch.empty((M, N), dtype=_out_dtype(cfg.y_dtype), device=x.device)
    _check("mxfp4_linear_fwd_save", lib().mxfp4_linear_fwd_save(
        _ptr(x), _ptr(w), _ptr(y), M, N, K, ctypes.byref(cfg), _ptr(workspace), workspace.numel(), _ptr(saved),
        saved.numel(), _stream_ptr(stream)))
    return y, workspace, saved


def mxfp4_linear_bwd_saved(dy, saved, K: int, cfg: LinearCfg, dx=None, dw=None, need_dx: bool = True,
                           need_dw: bool = True, workspace=None, stream=None):
    """Dgrad and Wgrad against the operands mxfp4_linear_fwd_save left in `saved`.  Returns (dx, dw, workspace)."""
    import torch
    M, N = dy.shape
    assert dy.is_contiguous()
    if workspace is None:
        workspace = torch.empty(mxfp4_linear_workspace_bytes(M, N, K, cfg, True), dtype=torch.uint8, device=dy.device)
    if need_dx and dx is None:
        dx = torch.empty((M, K), dtype=_out_dtype(cfg.dx_dtype), device=dy.device)
    if need_dw and dw is None:
        assert not cfg.dw_accumulate, "accumulating into dW needs the caller's dW"
        dw = torch.empty((N, K), dtype=_out_dtype(cfg.dw_dtype), device=dy.device)
    _check("mxfp4_linear_bwd_saved", lib().mxfp4_linear_bwd_saved(
        _ptr(dy), _ptr(saved), saved.numel(), _ptr(dx) if need_dx else None, _ptr(dw) if need_dw else None, M, N, K,
        ctypes.byref(cfg), _ptr(workspace), workspace.numel(), _stream_ptr(stream)))
    return dx, dw, workspace

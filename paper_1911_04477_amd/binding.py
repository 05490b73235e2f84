"""Thin ctypes binding of libbnn.so: argument marshalling only.

Every function takes torch tensors that already live on the GPU, passes their
data pointers, sizes and the current HIP stream to the C entry point of the same
name, and raises ``BnnError`` on a non-zero status.  No arithmetic of the method
happens in Python, and there is no CPU fallback: if the HIP library has not been
built, loading fails loudly.
"""
from __future__ import annotations

import ctypes
import importlib.util
import os
import warnings
from typing import List, Optional, Tuple

import torch

from .build import tensorcall_built_for

HERE = os.path.dirname(os.path.abspath(__file__))
# BNN_SANITIZE=1 (host-only checks, see build.py): the build whose host code carries ASan / UBSan
LIB_PATH = os.path.join(HERE, "libbnn_san.so" if os.environ.get("BNN_SANITIZE") == "1" else "libbnn.so")

_i64, _i32, _p, _sz = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t


class ChainLayer(ctypes.Structure):
    """bnn_chain_layer"""
    _fields_ = [("w_chain", _p), ("scale", _p), ("bias", _p), ("D", _i32), ("pool", _i32)]


# name -> (restype, argtypes); the list mirrors include/bnn.h one to one.
SIGNATURES = {
    "bnn_status_str": (ctypes.c_char_p, [_i32]),
    "bnn_packed_words": (_i64, [_i64]),
    "bnn_conv_kwords": (_i64, [_i32, _i32, _i32]),
    "bnn_conv_out_dim": (_i64, [_i64, _i64, _i64, _i64]),
    "bnn_encode": (_i32, [_p, _i64, _i64, _i64, _p, _i64, _p]),
    "bnn_pack_conv_weight": (_i32, [_p, _i32, _i32, _i32, _i32, _p, _p]),
    "bnn_im2col_packed": (_i32, [_p] + [_i32] * 10 + [_p, _p, _sz, _p]),
    "bnn_im2col_workspace_bytes": (_sz, [_i32] * 10),
    "bnn_xnor_gemm": (_i32, [_p, _i64, _p, _i64, _p, _i64, _i64, _i64, _i64, _p]),
    "bnn_xnor_gemm_mfma_i8": (_i32, [_p, _i64, _p, _i64, _p, _i64, _i64, _i64, _i64, _p]),
    "bnn_xnor_gemm_mfma_fp4": (_i32, [_p, _i64, _p, _i64, _p, _i64, _i64, _i64, _i64, _p]),
    "bnn_fp4_row_bytes": (_i64, [_i64]),
    "bnn_expand_fp4": (_i32, [_p, _i64, _i64, _i64, _p, _i64, _p]),
    "bnn_xnor_gemm_mfma_fp4_expanded": (_i32, [_p, _i64, _p, _i64, _p, _i64, _i64, _i64, _i64, _p]),
    "bnn_conv2d_mfma_fp4_expanded": (_i32, [_p, _p] + [_i32] * 11 + [_p, _p]),
    "bnn_control_conv2d_f32": (_i32, [_p, _p] + [_i32] * 11 + [_p, _p]),
    "bnn_xnor_gemm_epilogue": (_i32, [_p, _i64, _p, _i64, _i64, _i64, _i64, _p, _i64, _p, _i64, _p, _p, _i32, _p]),
    "bnn_conv2d": (_i32, [_p, _p] + [_i32] * 11 + [_p, _p, _p, _p, _p, _sz, _p]),
    "bnn_conv2d_workspace_bytes": (_sz, [_i32] * 10),
    "bnn_conv2d_noalloc": (_i32, [_p, _p] + [_i32] * 11 + [_p, _p, _p, _p, _p]),
    "bnn_conv2d_noalloc_max_bytes": (_sz, []),
    "bnn_conv2d_packed": (_i32, [_p, _p] + [_i32] * 12 + [_p, _p, _p, _p, _p, _p]),
    "bnn_conv_chain_weight_bytes": (_sz, [_i32, _i32]),
    "bnn_pack_conv_chain_weight": (_i32, [_p, _i32, _i32, _p, _p]),
    "bnn_conv_chain_pays": (_i32, [_i32] * 5 + [ctypes.POINTER(ChainLayer)]),
    "bnn_conv_chain": (_i32, [_p] + [_i32] * 5 + [ctypes.POINTER(ChainLayer), _p, _p]),
    "bnn_conv2d_f32_sign": (_i32, [_p, _p] + [_i32] * 11 + [_p, _p, _p, _p]),
    "bnn_pack_fc_weight_nhwc": (_i32, [_p, _i64, _i32, _i32, _i32, _p, _p]),
    "bnn_maxpool2x2": (_i32, [_p, _i32, _i32, _i32, _i32, _p, _p, _p, _p, _p]),
    "bnn_conv2d_f32": (_i32, [_p, _p] + [_i32] * 11 + [_p, _p, _p, _p]),
    "bnn_fc_f32": (_i32, [_p, _p, _p, _i64, _i64, _i64, _i32, _p, _p]),
}

# include/bnn_testing.h: the same calls with the kernel variant chosen by the caller, the
# kernel-timing hook and the two yardstick kernels.  Tests and bench.py only.
TESTING_SIGNATURES = {
    "bnn_testing_xnor_gemm_epilogue": (_i32, [_p, _i64, _p, _i64, _i64, _i64, _i64, _p, _i64, _p, _i64, _p, _p, _i32,
                                              _i32, _p]),
    "bnn_testing_conv2d": (_i32, [_p, _p] + [_i32] * 11 + [_p, _p, _p, _p, _p, _sz, _i32, _i32, _p]),
    "bnn_testing_conv2d_packed": (_i32, [_p, _p] + [_i32] * 12 + [_p, _p, _p, _p, _p, _i32, _i32, _p]),
    "bnn_testing_conv_image": (_i32, [_i32] * 14 + [ctypes.POINTER(_i64)]),
    "bnn_testing_conv_word": (_i32, [_i32] * 14),
    "bnn_testing_conv_word_nontemporal": (_i32, [_i32] * 11),
    "bnn_testing_first_sign": (_i32, [_i32] * 9),
    "bnn_testing_conv_region": (_i32, [_i32] * 12 + [ctypes.POINTER(_i64)]),
    "bnn_testing_nontemporal_maps": (_i32, [_i32, _i32, _i32, _i64, _i64]),
    "bnn_testing_xnor_gemm_mfma_fp4_expanded": (_i32, [_p, _i64, _p, _i64, _p, _i64, _i64, _i64, _i64, _i32, _p]),
    "bnn_prof_enable": (_i32, [_i32]),
    "bnn_prof_reset": (_i32, []),
    "bnn_prof_count": (_i64, []),
    "bnn_prof_get": (_i32, [_i64, ctypes.POINTER(_i32), ctypes.POINTER(ctypes.c_float)]),
    "bnn_kernel_name": (ctypes.c_char_p, [_i32]),
    "bnn_valu_peak_probe": (_i32, [_p, _i32, _i32, _i32, _p]),
    "bnn_copy_probe": (_i32, [_p, _p, _sz, _p]),
}

BNN_OK = 0
CH_NONE, CH_ROW, CH_COL = 0, 1, 2

_lib: Optional[ctypes.CDLL] = None


FASTCALL_PATH = LIB_PATH.replace("libbnn", "_fastcall")
TENSORCALL_PATH = LIB_PATH.replace("libbnn", "_tensorcall")


def _fastcall():
    """The call helper, or None (with a warning) where only libbnn has been built."""
    if not os.path.exists(FASTCALL_PATH):
        warnings.warn(f"{FASTCALL_PATH} is missing: build it with `python paper_1911_04477_amd/build.py`; until then calls "
                      "go through ctypes, 0.4 to 0.9 us slower each", RuntimeWarning, stacklevel=4)
        return None
    spec = importlib.util.spec_from_file_location("paper_1911_04477_amd._fastcall", FASTCALL_PATH)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


class _Calls:
    """The functions of SIGNATURES and TESTING_SIGNATURES whose arguments are integers and raw pointers, called without
    ctypes' conversions (csrc/fastcall.c)."""

    _KINDS = {_p: "p", _i64: "q", _i32: "i", _sz: "z"}

    def __init__(self, L: ctypes.CDLL):
        fast = _fastcall()
        for name, (res, args) in list(SIGNATURES.items()) + list(TESTING_SIGNATURES.items()):
            args = [_p if isinstance(a, type) and issubclass(a, ctypes._Pointer) else a for a in args]
            if res not in (_i32, _i64, _sz) or any(a not in self._KINDS for a in args):
                continue
            address = ctypes.cast(getattr(L, name), ctypes.c_void_p).value
            setattr(self, name, fast.Function(address, "".join(self._KINDS[a] for a in args), "i" if res is _i32 else "q")
                    if fast else ctypes.CFUNCTYPE(res, *args)(address))


_calls: Optional[_Calls] = None


def _c() -> _Calls:
    global _calls
    if _calls is None:
        _calls = _Calls(lib())
    return _calls


class _Tensors:
    """Calls from the tensors themselves (csrc/tensorcall.cpp): a status, or None where the call is not a plain one and the
    function of this module has to look at it.  Where the extension has not been built, or for another torch, every call is of that
    kind."""

    FUNCTIONS = ("gemm", "epilogue", "encode", "conv2d", "conv2d_packed", "im2col", "f32_sign", "conv2d_f32", "maxpool", "fc")

    def __init__(self, L: ctypes.CDLL, path: str):
        module = None
        if os.path.exists(path):
            try:
                spec = importlib.util.spec_from_file_location("paper_1911_04477_amd._tensorcall", path)
                module = importlib.util.module_from_spec(spec)
                spec.loader.exec_module(module)
                if module.built_for != tensorcall_built_for(torch):  # it would read tensors at wrong places
                    raise ImportError(f"built for {module.built_for}")
            except (ImportError, AttributeError) as e:  # of another torch or Python
                module = None
                warnings.warn(f"{path} does not load ({e}): build it again; calls take 1 to 2 us longer", RuntimeWarning, stacklevel=4)
        if module is not None:
            module.bind(*[ctypes.cast(getattr(L, name), ctypes.c_void_p).value for name in module.names])
        for f in self.FUNCTIONS:
            setattr(self, f, getattr(module, f) if module is not None else lambda *args: None)


_tensors: Optional[_Tensors] = None


def _t() -> _Tensors:
    global _tensors
    if _tensors is None:
        _tensors = _Tensors(lib(), TENSORCALL_PATH)
    return _tensors


class BnnError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = int(status)
        name = lib().bnn_status_str(self.status).decode()
        super().__init__(f"{where} failed: {name} ({self.status})")


def lib() -> ctypes.CDLL:
    """Load libbnn.so (built by paper_1911_04477_amd/build.py).  No fallback."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                f"{LIB_PATH} is missing: build it with `python paper_1911_04477_amd/build.py` "
                "(there is no CPU fallback)")
        L = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in list(SIGNATURES.items()) + list(TESTING_SIGNATURES.items()):
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        _lib = L
    return _lib


def _check(st: int, where: str) -> None:
    if st != BNN_OK:
        raise BnnError(st, where)


def _stream() -> int:
    # the current stream of the current device as a raw handle: torch.cuda.current_stream() builds a Stream object
    # on every call, 2.7 of the 8.4 us that a whole call through this binding took (0.1 us this way)
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())


def _ptr(t: Optional[torch.Tensor]) -> Optional[int]:
    return None if t is None else t.data_ptr()


def _dev(t: torch.Tensor, dtype: torch.dtype, name: str) -> None:
    if not t.is_cuda or t.dtype != dtype:
        raise TypeError(f"{name} must be a GPU tensor of dtype {dtype}")


def packed_words(K: int) -> int:
    return _c().bnn_packed_words(K)


def conv_kwords(C: int, kH: int, kW: int) -> int:
    return int(_c().bnn_conv_kwords(C, kH, kW))


def conv_out_dim(n: int, k: int, s: int, p: int) -> int:
    return int(_c().bnn_conv_out_dim(n, k, s, p))


def bnn_encode(src: torch.Tensor, dst: Optional[torch.Tensor] = None) -> torch.Tensor:
    """src fp32 [rows, K] (row stride = src.stride(0)) -> int64-typed packed words [rows, Kw]."""
    if dst is not None:
        st = _t().encode(src, dst)
        if st is not None:
            _check(st, "bnn_encode")
            return dst
    _dev(src, torch.float32, "src")
    assert src.dim() == 2 and src.stride(1) == 1
    rows, K = src.shape
    Kw = packed_words(K)
    if dst is None:
        dst = torch.empty((rows, Kw), dtype=torch.int64, device=src.device)
    _dev(dst, torch.int64, "dst")
    assert dst.stride(1) == 1
    _check(_c().bnn_encode(_ptr(src), rows, K, src.stride(0) if rows > 1 else max(K, src.stride(0)), _ptr(dst),
                            dst.stride(0) if rows > 1 else max(Kw, dst.stride(0)), _stream()), "bnn_encode")
    return dst


def bnn_pack_conv_weight(w: torch.Tensor) -> torch.Tensor:
    _dev(w, torch.float32, "w")
    assert w.dim() == 4 and w.is_contiguous()
    D, C, kH, kW = w.shape
    out = torch.empty((D, conv_kwords(C, kH, kW)), dtype=torch.int64, device=w.device)
    _check(_c().bnn_pack_conv_weight(_ptr(w), D, C, kH, kW, _ptr(out), _stream()), "bnn_pack_conv_weight")
    return out


def im2col_workspace_bytes(x_shape, kH, kW, stride, pad) -> int:
    N, C, H, W = x_shape
    return int(_c().bnn_im2col_workspace_bytes(N, C, H, W, kH, kW, stride[0], stride[1], pad[0], pad[1]))


def bnn_im2col_packed(x: torch.Tensor, kH: int, kW: int, stride=(1, 1), pad=(0, 0),
                      cols: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    if cols is not None and workspace is not None:
        st = _t().im2col(x, kH, kW, stride, pad, cols, workspace)
        if st is not None:
            _check(st, "bnn_im2col_packed")
            return cols
    _dev(x, torch.float32, "x")
    assert x.dim() == 4 and x.is_contiguous()
    N, C, H, W = x.shape
    geo = (N, C, H, W, kH, kW, stride[0], stride[1], pad[0], pad[1])
    OH, OW = conv_out_dim(H, kH, stride[0], pad[0]), conv_out_dim(W, kW, stride[1], pad[1])
    if cols is None:
        cols = torch.empty((N * OH * OW, conv_kwords(C, kH, kW)), dtype=torch.int64, device=x.device)
    _dev(cols, torch.int64, "cols")
    assert cols.is_contiguous() and cols.numel() == N * OH * OW * conv_kwords(C, kH, kW)
    nbytes = int(_c().bnn_im2col_workspace_bytes(*geo))
    if workspace is None:
        workspace = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=x.device)
    _check(_c().bnn_im2col_packed(_ptr(x), *geo, _ptr(cols), _ptr(workspace), workspace.numel(), _stream()),
           "bnn_im2col_packed")
    return cols


def bnn_xnor_gemm(A: torch.Tensor, B: torch.Tensor, K: int, C: Optional[torch.Tensor] = None,
                  cfg: Optional[int] = None) -> torch.Tensor:
    """A [M, >=Kw], B [N, >=Kw] packed (int64-typed) -> int32 [M, N].
    cfg (tests only): the same call through bnn_testing_xnor_gemm_epilogue on that tile configuration."""
    if C is not None and cfg is None:
        st = _t().gemm(A, B, K, C)
        if st is not None:
            _check(st, "bnn_xnor_gemm")
            return C
    _dev(A, torch.int64, "A")
    _dev(B, torch.int64, "B")
    M, N = A.shape[0], B.shape[0]
    if C is None:
        C = torch.empty((M, N), dtype=torch.int32, device=A.device)
    _dev(C, torch.int32, "C")
    lda = A.stride(0) if M > 1 else max(A.shape[1], 1)
    ldb = B.stride(0) if N > 1 else max(B.shape[1], 1)
    ldc = C.stride(0) if M > 1 else max(N, 1)
    if cfg is None:
        _check(_c().bnn_xnor_gemm(_ptr(A), lda, _ptr(B), ldb, _ptr(C), ldc, M, N, K, _stream()), "bnn_xnor_gemm")
    else:
        _check(_c().bnn_testing_xnor_gemm_epilogue(_ptr(A), lda, _ptr(B), ldb, M, N, K, _ptr(C), ldc, None, 0, None,
                                                    None, CH_NONE, cfg, _stream()), "bnn_testing_xnor_gemm_epilogue")
    return C


def bnn_xnor_gemm_mfma_i8(A: torch.Tensor, B: torch.Tensor, K: int, C: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Ablation: same contract as bnn_xnor_gemm, computed with int8 MFMA."""
    _dev(A, torch.int64, "A")
    _dev(B, torch.int64, "B")
    M, N = A.shape[0], B.shape[0]
    if C is None:
        C = torch.empty((M, N), dtype=torch.int32, device=A.device)
    lda = A.stride(0) if M > 1 else max(A.shape[1], 1)
    ldb = B.stride(0) if N > 1 else max(B.shape[1], 1)
    _check(_c().bnn_xnor_gemm_mfma_i8(_ptr(A), lda, _ptr(B), ldb, _ptr(C), C.stride(0) if M > 1 else max(N, 1), M, N,
                                       K, _stream()), "bnn_xnor_gemm_mfma_i8")
    return C


def bnn_xnor_gemm_mfma_fp4(A: torch.Tensor, B: torch.Tensor, K: int, C: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Ablation: same contract as bnn_xnor_gemm, computed with the 4-bit floating-point MFMA."""
    _dev(A, torch.int64, "A")
    _dev(B, torch.int64, "B")
    M, N = A.shape[0], B.shape[0]
    if C is None:
        C = torch.empty((M, N), dtype=torch.int32, device=A.device)
    lda = A.stride(0) if M > 1 else max(A.shape[1], 1)
    ldb = B.stride(0) if N > 1 else max(B.shape[1], 1)
    _check(_c().bnn_xnor_gemm_mfma_fp4(_ptr(A), lda, _ptr(B), ldb, _ptr(C), C.stride(0) if M > 1 else max(N, 1), M, N,
                                        K, _stream()), "bnn_xnor_gemm_mfma_fp4")
    return C


def bnn_expand_fp4(packed: torch.Tensor, K: int, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Ablation: packed sign rows [rows, >= ceil(K/64)] int64 -> E2M1 rows [rows, 32 * ceil(K/64)] uint8."""
    _dev(packed, torch.int64, "packed")
    rows = packed.shape[0]
    rb = int(_c().bnn_fp4_row_bytes(K))
    if out is None:
        out = torch.empty((rows, rb), dtype=torch.uint8, device=packed.device)
    src_ld = packed.stride(0) if rows > 1 else max(packed.shape[1], 1)
    dst_ld = out.stride(0) if rows > 1 else max(out.shape[1], 16)
    _check(_c().bnn_expand_fp4(_ptr(packed), rows, K, src_ld, _ptr(out), dst_ld, _stream()), "bnn_expand_fp4")
    return out


def bnn_xnor_gemm_mfma_fp4_expanded(A4: torch.Tensor, B4: torch.Tensor, K: int, C: Optional[torch.Tensor] = None,
                                    tile: Optional[int] = None) -> torch.Tensor:
    """Ablation: the binarized GEMM on operands kept in memory as E2M1 +-1 rows (bnn_expand_fp4)."""
    _dev(A4, torch.uint8, "A4")
    _dev(B4, torch.uint8, "B4")
    M, N = A4.shape[0], B4.shape[0]
    if C is None:
        C = torch.empty((M, N), dtype=torch.int32, device=A4.device)
    lda = A4.stride(0) if M > 1 else max(A4.shape[1], 16)
    ldb = B4.stride(0) if N > 1 else max(B4.shape[1], 16)
    ldc = C.stride(0) if M > 1 else max(N, 1)
    if tile is None:
        _check(_c().bnn_xnor_gemm_mfma_fp4_expanded(_ptr(A4), lda, _ptr(B4), ldb, _ptr(C), ldc, M, N, K, _stream()),
               "bnn_xnor_gemm_mfma_fp4_expanded")
    else:
        _check(_c().bnn_testing_xnor_gemm_mfma_fp4_expanded(_ptr(A4), lda, _ptr(B4), ldb, _ptr(C), ldc, M, N, K, tile,
                                                             _stream()), "bnn_testing_xnor_gemm_mfma_fp4_expanded")
    return C


def bnn_conv2d_mfma_fp4_expanded(x4: torch.Tensor, w4: torch.Tensor, C: int, D: int, kH: int, kW: int, stride=(1, 1),
                                 pad=(0, 0), out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Ablation: x4 [N, H, W, C/2] uint8 (E2M1 codes), w4 [D, kH*kW*C/2] uint8 -> int32 NCHW."""
    _dev(x4, torch.uint8, "x4")
    _dev(w4, torch.uint8, "w4")
    assert x4.dim() == 4 and x4.is_contiguous() and w4.is_contiguous()
    N, H, W, _ = x4.shape
    OH, OW = conv_out_dim(H, kH, stride[0], pad[0]), conv_out_dim(W, kW, stride[1], pad[1])
    if out is None:
        out = torch.empty((N, D, OH, OW), dtype=torch.int32, device=x4.device)
    _check(_c().bnn_conv2d_mfma_fp4_expanded(_ptr(x4), _ptr(w4), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0],
                                              pad[1], _ptr(out), _stream()), "bnn_conv2d_mfma_fp4_expanded")
    return out


def bnn_control_conv2d_f32(x: torch.Tensor, w: torch.Tensor, stride=(1, 1), pad=(0, 0),
                           out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Control group: the binarized convolution as an fp32 GEMM on sign(x), sign(w)."""
    _dev(x, torch.float32, "x")
    _dev(w, torch.float32, "w")
    N, C, H, W = x.shape
    D, _, kH, kW = w.shape
    OH, OW = conv_out_dim(H, kH, stride[0], pad[0]), conv_out_dim(W, kW, stride[1], pad[1])
    if out is None:
        out = torch.empty((N, D, OH, OW), dtype=torch.float32, device=x.device)
    _check(_c().bnn_control_conv2d_f32(_ptr(x), _ptr(w), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0], pad[1],
                                        _ptr(out), _stream()), "bnn_control_conv2d_f32")
    return out


def bnn_xnor_gemm_epilogue(A: torch.Tensor, B: torch.Tensor, K: int, scale: torch.Tensor, bias: torch.Tensor,
                           axis: int, want_int: bool = False, out_y: Optional[torch.Tensor] = None,
                           cfg: Optional[int] = None) -> Tuple[Optional[torch.Tensor], torch.Tensor]:
    if out_y is not None and not want_int and cfg is None:
        st = _t().epilogue(A, B, K, scale, bias, axis, out_y)
        if st is not None:
            _check(st, "bnn_xnor_gemm_epilogue")
            return None, out_y
    _dev(A, torch.int64, "A")
    _dev(B, torch.int64, "B")
    M, N = A.shape[0], B.shape[0]
    if out_y is not None:
        _dev(out_y, torch.float32, "out_y")
        assert out_y.shape == (M, N) and out_y.is_contiguous()
    Y = out_y if out_y is not None else torch.empty((M, N), dtype=torch.float32, device=A.device)
    C = torch.empty((M, N), dtype=torch.int32, device=A.device) if want_int else None
    lda = A.stride(0) if M > 1 else max(A.shape[1], 1)
    ldb = B.stride(0) if N > 1 else max(B.shape[1], 1)
    if cfg is None:
        _check(_c().bnn_xnor_gemm_epilogue(_ptr(A), lda, _ptr(B), ldb, M, N, K, _ptr(C), max(N, 1), _ptr(Y), max(N, 1),
                                            _ptr(scale), _ptr(bias), axis, _stream()), "bnn_xnor_gemm_epilogue")
    else:
        _check(_c().bnn_testing_xnor_gemm_epilogue(_ptr(A), lda, _ptr(B), ldb, M, N, K, _ptr(C), max(N, 1), _ptr(Y),
                                                    max(N, 1), _ptr(scale), _ptr(bias), axis, cfg, _stream()),
               "bnn_testing_xnor_gemm_epilogue")
    return C, Y


def conv2d_workspace_bytes(x_shape, kH, kW, stride, pad) -> int:
    N, C, H, W = x_shape
    return int(_c().bnn_conv2d_workspace_bytes(N, C, H, W, kH, kW, stride[0], stride[1], pad[0], pad[1]))


def bnn_conv2d(x: torch.Tensor, w_packed: torch.Tensor, D: int, kH: int, kW: int, stride=(1, 1), pad=(0, 0),
               scale: Optional[torch.Tensor] = None, bias: Optional[torch.Tensor] = None, want_int: bool = True,
               workspace: Optional[torch.Tensor] = None, out_i32: Optional[torch.Tensor] = None,
               out_f32: Optional[torch.Tensor] = None, cfg: Optional[int] = None, lean: Optional[int] = None):
    """Returns (out_i32 or None, out_f32 or None), both NCHW.
    cfg / lean (tests only): the same call through bnn_testing_conv2d."""
    if (workspace is not None and (out_i32 is not None or not want_int) and (out_f32 is not None or scale is None)
            and cfg is None and lean is None):
        st = _t().conv2d(x, w_packed, D, kH, kW, stride, pad, out_i32, out_f32, scale, bias, workspace)
        if st is not None:
            _check(st, "bnn_conv2d")
            return out_i32, out_f32
    _dev(x, torch.float32, "x")
    _dev(w_packed, torch.int64, "w_packed")
    assert x.dim() == 4 and x.is_contiguous() and w_packed.is_contiguous()
    N, C, H, W = x.shape
    OH, OW = conv_out_dim(H, kH, stride[0], pad[0]), conv_out_dim(W, kW, stride[1], pad[1])
    nbytes = conv2d_workspace_bytes(x.shape, kH, kW, stride, pad)
    if workspace is None:
        workspace = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=x.device)
    if want_int and out_i32 is None:
        out_i32 = torch.empty((N, D, OH, OW), dtype=torch.int32, device=x.device)
    if scale is not None and out_f32 is None:
        out_f32 = torch.empty((N, D, OH, OW), dtype=torch.float32, device=x.device)
    if cfg is None and lean is None:
        _check(_c().bnn_conv2d(_ptr(x), _ptr(w_packed), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0], pad[1],
                                _ptr(out_i32), _ptr(out_f32), _ptr(scale), _ptr(bias), _ptr(workspace),
                                workspace.numel(), _stream()), "bnn_conv2d")
    else:
        _check(_c().bnn_testing_conv2d(_ptr(x), _ptr(w_packed), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0],
                                        pad[1], _ptr(out_i32), _ptr(out_f32), _ptr(scale), _ptr(bias),
                                        _ptr(workspace), workspace.numel(), -1 if cfg is None else cfg,
                                        1 if lean is None else lean, _stream()), "bnn_testing_conv2d")
    return out_i32, out_f32


def bnn_conv2d_noalloc(x: torch.Tensor, w_packed: torch.Tensor, D: int, kH: int, kW: int, stride, pad,
                       out_i32: Optional[torch.Tensor], out_f32: Optional[torch.Tensor] = None,
                       scale: Optional[torch.Tensor] = None, bias: Optional[torch.Tensor] = None) -> None:
    """bnn_conv2d without a workspace argument; the caller passes every output buffer, so the call
    allocates nothing on either side of the ABI."""
    _dev(x, torch.float32, "x")
    _dev(w_packed, torch.int64, "w_packed")
    assert x.dim() == 4 and x.is_contiguous() and w_packed.is_contiguous()
    N, C, H, W = x.shape
    _check(_c().bnn_conv2d_noalloc(_ptr(x), _ptr(w_packed), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0],
                                    pad[1], _ptr(out_i32), _ptr(out_f32), _ptr(scale), _ptr(bias), _stream()),
           "bnn_conv2d_noalloc")


def bnn_conv2d_packed(xp: torch.Tensor, w_packed: torch.Tensor, C: int, D: int, kH: int, kW: int, stride=(1, 1),
                      pad=(0, 0), pool: int = 0, scale: Optional[torch.Tensor] = None,
                      bias: Optional[torch.Tensor] = None, out: str = "packed", out_buf: Optional[torch.Tensor] = None,
                      cfg: Optional[int] = None, lean: Optional[int] = None):
    """xp: packed NHWC [N, H, W, Cw] (int64-typed).  out = "packed" | "i32" | "f32".
    cfg / lean (tests only): the same call through bnn_testing_conv2d_packed."""
    if out_buf is not None and cfg is None and lean is None and out in ("packed", "i32", "f32"):
        st = _t().conv2d_packed(xp, w_packed, C, D, kH, kW, stride, pad, pool, out_buf if out == "i32" else None,
                                out_buf if out == "f32" else None, out_buf if out == "packed" else None, scale, bias)
        if st is not None:
            _check(st, "bnn_conv2d_packed")
            return out_buf
    _dev(xp, torch.int64, "x_packed")
    _dev(w_packed, torch.int64, "w_packed")
    assert xp.dim() == 4 and xp.is_contiguous() and w_packed.is_contiguous()
    N, H, W, Cw = xp.shape
    assert Cw == packed_words(C)
    OH, OW = conv_out_dim(H, kH, stride[0], pad[0]), conv_out_dim(W, kW, stride[1], pad[1])
    oi = of = op = None
    if out == "packed":
        op = out_buf if out_buf is not None else torch.empty(
            (N, OH // 2 if pool else OH, OW // 2 if pool else OW, packed_words(D)), dtype=torch.int64, device=xp.device)
    elif out == "i32":
        oi = out_buf if out_buf is not None else torch.empty((N, D, OH, OW), dtype=torch.int32, device=xp.device)
    elif out == "f32":
        of = out_buf if out_buf is not None else torch.empty((N, D, OH, OW), dtype=torch.float32, device=xp.device)
    else:
        raise ValueError(out)
    if cfg is None and lean is None:
        _check(_c().bnn_conv2d_packed(_ptr(xp), _ptr(w_packed), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0],
                                       pad[1], pool, _ptr(oi), _ptr(of), _ptr(op), _ptr(scale), _ptr(bias), _stream()),
               "bnn_conv2d_packed")
    else:
        _check(_c().bnn_testing_conv2d_packed(_ptr(xp), _ptr(w_packed), N, C, H, W, D, kH, kW, stride[0], stride[1],
                                               pad[0], pad[1], pool, _ptr(oi), _ptr(of), _ptr(op), _ptr(scale),
                                               _ptr(bias), -1 if cfg is None else cfg, 1 if lean is None else lean,
                                               _stream()), "bnn_testing_conv2d_packed")
    return op if op is not None else (oi if oi is not None else of)


def bnn_pack_conv_chain_weight(w_packed: torch.Tensor, C: int, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Filter bank of a 3x3 layer from bnn_pack_conv_weight, in the order in which bnn_conv_chain multiplies it."""
    _dev(w_packed, torch.int64, "w_packed")
    D = w_packed.shape[0]
    assert w_packed.is_contiguous() and w_packed.shape[1] == conv_kwords(C, 3, 3)
    if out is None:
        out = torch.empty(max(16, int(_c().bnn_conv_chain_weight_bytes(C, D))), dtype=torch.uint8, device=w_packed.device)
    else:
        _chain_weight(out, C, D)
    _check(_c().bnn_pack_conv_chain_weight(_ptr(w_packed), D, C, _ptr(out), _stream()), "bnn_pack_conv_chain_weight")
    return out


def _chain_weight(w: torch.Tensor, C: int, D: int) -> None:
    _dev(w, torch.uint8, "w_chain")
    need = int(_c().bnn_conv_chain_weight_bytes(C, D))
    if not w.is_contiguous() or w.numel() < need:
        raise ValueError(f"w_chain: {need} contiguous bytes for {C} to {D} channels")


def conv_chain_layers(layers) -> ctypes.Array:
    """[(w_chain or None, scale, bias, D, pool)] -> the host array bnn_conv_chain takes.  It holds the tensors whose
    addresses it contains (`tensors`), so they live as long as it does.  w_chain None: for bnn_conv_chain_pays alone."""
    layers = [tuple(L) for L in layers]
    for i, (w, s, b, D, pool) in enumerate(layers):
        for t, name in ((s, "scale"), (b, "bias")):
            _dev(t, torch.float32, name)
            if not t.is_contiguous() or t.numel() < D:
                raise ValueError(f"{name}: {D} contiguous values")
        if w is not None and i > 0:  # the first layer's: where its input channels are known
            _chain_weight(w, layers[i - 1][3], D)
    out = (ChainLayer * len(layers))(*[ChainLayer(_ptr(w), _ptr(s), _ptr(b), D, pool) for w, s, b, D, pool in layers])
    out.tensors = [L[:3] for L in layers]
    return out


def bnn_conv_chain_pays(N: int, C: int, H: int, W: int, layers: ctypes.Array) -> bool:
    return bool(_c().bnn_conv_chain_pays(N, C, H, W, len(layers), ctypes.addressof(layers)))


def bnn_conv_chain(xp: torch.Tensor, C: int, layers: ctypes.Array, out: torch.Tensor) -> torch.Tensor:
    """xp: packed NHWC [N, H, W, C / 64] through consecutive 3x3 layers; out: the last layer's packed map."""
    _dev(xp, torch.int64, "x_packed")
    _dev(out, torch.int64, "out")
    N, H, W, Cw = xp.shape
    assert xp.is_contiguous() and out.is_contiguous() and Cw == packed_words(C)
    held = getattr(layers, "tensors", None)  # an array of another origin is the caller's own
    if held and held[0][0] is not None:
        _chain_weight(held[0][0], C, layers[0].D)
    OH, OW = H, W
    for L in layers:
        if L.pool:
            OH, OW = OH // 2, OW // 2
    assert tuple(out.shape) == (N, OH, OW, packed_words(layers[-1].D))
    _check(_c().bnn_conv_chain(_ptr(xp), N, C, H, W, len(layers), ctypes.addressof(layers), _ptr(out), _stream()), "bnn_conv_chain")
    return out


def bnn_conv2d_f32_sign(x: torch.Tensor, w: torch.Tensor, scale: torch.Tensor, bias: torch.Tensor, stride=(1, 1),
                        pad=(0, 0), out: Optional[torch.Tensor] = None) -> torch.Tensor:
    if out is not None:
        st = _t().f32_sign(x, w, scale, bias, stride, pad, out)
        if st is not None:
            _check(st, "bnn_conv2d_f32_sign")
            return out
    _dev(x, torch.float32, "x")
    _dev(w, torch.float32, "w")
    N, C, H, W = x.shape
    D, _, kH, kW = w.shape
    OH, OW = conv_out_dim(H, kH, stride[0], pad[0]), conv_out_dim(W, kW, stride[1], pad[1])
    if out is None:
        out = torch.empty((N, OH, OW, packed_words(D)), dtype=torch.int64, device=x.device)
    _check(_c().bnn_conv2d_f32_sign(_ptr(x), _ptr(w), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0], pad[1],
                                     _ptr(scale), _ptr(bias), _ptr(out), _stream()), "bnn_conv2d_f32_sign")
    return out


def bnn_pack_fc_weight_nhwc(w: torch.Tensor, C: int, H: int, W: int) -> torch.Tensor:
    _dev(w, torch.float32, "w")
    assert w.dim() == 2 and w.is_contiguous() and w.shape[1] == C * H * W
    out = torch.empty((w.shape[0], H * W * packed_words(C)), dtype=torch.int64, device=w.device)
    _check(_c().bnn_pack_fc_weight_nhwc(_ptr(w), w.shape[0], C, H, W, _ptr(out), _stream()),
           "bnn_pack_fc_weight_nhwc")
    return out


def bnn_maxpool2x2(a: torch.Tensor, scale: Optional[torch.Tensor] = None, bias: Optional[torch.Tensor] = None,
                   want_int: bool = True, out_i32=None, out_f32=None):
    if (out_i32 is not None or not want_int) and (out_f32 is not None or scale is None):
        st = _t().maxpool(a, out_i32, out_f32, scale, bias)
        if st is not None:
            _check(st, "bnn_maxpool2x2")
            return out_i32, out_f32
    _dev(a, torch.int32, "in")
    assert a.dim() == 4 and a.is_contiguous()
    N, D, H, W = a.shape
    if want_int and out_i32 is None:
        out_i32 = torch.empty((N, D, H // 2, W // 2), dtype=torch.int32, device=a.device)
    if scale is not None and out_f32 is None:
        out_f32 = torch.empty((N, D, H // 2, W // 2), dtype=torch.float32, device=a.device)
    _check(_c().bnn_maxpool2x2(_ptr(a), N, D, H, W, _ptr(out_i32), _ptr(out_f32), _ptr(scale), _ptr(bias),
                                _stream()), "bnn_maxpool2x2")
    return out_i32, out_f32


def bnn_conv2d_f32(x: torch.Tensor, w: torch.Tensor, stride=(1, 1), pad=(0, 0), scale=None, bias=None, out=None):
    if out is not None:
        st = _t().conv2d_f32(x, w, scale, bias, stride, pad, out)
        if st is not None:
            _check(st, "bnn_conv2d_f32")
            return out
    _dev(x, torch.float32, "x")
    _dev(w, torch.float32, "w")
    N, C, H, W = x.shape
    D, _, kH, kW = w.shape
    OH, OW = conv_out_dim(H, kH, stride[0], pad[0]), conv_out_dim(W, kW, stride[1], pad[1])
    if out is None:
        out = torch.empty((N, D, OH, OW), dtype=torch.float32, device=x.device)
    _check(_c().bnn_conv2d_f32(_ptr(x), _ptr(w), N, C, H, W, D, kH, kW, stride[0], stride[1], pad[0], pad[1],
                                _ptr(scale), _ptr(bias), _ptr(out), _stream()), "bnn_conv2d_f32")
    return out


def bnn_fc_f32(x: torch.Tensor, w: torch.Tensor, bias: Optional[torch.Tensor] = None, sign_input: bool = False,
               out=None):
    if out is not None:
        st = _t().fc(x, w, bias, int(sign_input), out)
        if st is not None:
            _check(st, "bnn_fc_f32")
            return out
    _dev(x, torch.float32, "x")
    _dev(w, torch.float32, "w")
    M, K = x.shape
    N = w.shape[0]
    if out is None:
        out = torch.empty((M, N), dtype=torch.float32, device=x.device)
    _check(_c().bnn_fc_f32(_ptr(x), _ptr(w), _ptr(bias), M, K, N, int(sign_input), _ptr(out), _stream()),
           "bnn_fc_f32")
    return out


# ---- measurement helpers (include/bnn_testing.h) -----------------------------------
def prof_enable(on: bool) -> None:
    _check(_c().bnn_prof_enable(int(on)), "bnn_prof_enable")


def prof_reset() -> None:
    _check(_c().bnn_prof_reset(), "bnn_prof_reset")


def prof_records() -> List[Tuple[str, float]]:
    """(kernel name, milliseconds) of every launch recorded since the last reset."""
    L = lib()
    out = []
    kid, ms = _i32(0), ctypes.c_float(0.0)
    for i in range(int(L.bnn_prof_count())):
        _check(L.bnn_prof_get(i, ctypes.byref(kid), ctypes.byref(ms)), "bnn_prof_get")
        out.append((L.bnn_kernel_name(kid.value).decode(), float(ms.value)))
    return out


def bnn_valu_peak_probe(sink: torch.Tensor, blocks: int, iters: int, kind: int = 0) -> None:
    _dev(sink, torch.int32, "sink")
    assert sink.numel() >= blocks * 256
    _check(_c().bnn_valu_peak_probe(_ptr(sink), blocks, iters, kind, _stream()), "bnn_valu_peak_probe")


def bnn_copy_probe(src: torch.Tensor, dst: torch.Tensor) -> None:
    nbytes = src.numel() * src.element_size()
    assert dst.numel() * dst.element_size() >= nbytes
    _check(_c().bnn_copy_probe(_ptr(src), _ptr(dst), nbytes, _stream()), "bnn_copy_probe")

"""Thin Python binding of the C-ABI library libvidiq.so (declared in include/vq.h).

Argument marshalling only: torch supplies device memory and the current HIP
stream, every step of the quantized linear layer runs in the library's kernels.
Tensors are checked and turned into pointers in csrc/vq_torch.cpp (in Python it
took longer than a small layer runs on the device).  There is no fallback: if
the library is missing or a call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes
import importlib.machinery
import importlib.util
import os
import re

import torch

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
# the in-tree build; VQ_LIBVIDIQ_PATH names another build of the same sources (e.g. one with host sanitizers)
LIB_PATH = os.environ.get("VQ_LIBVIDIQ_PATH") or os.path.join(PKG_DIR, "libvidiq.so")
EXT_PATH = os.path.join(PKG_DIR, "_vq_torch.so")  # csrc/vq_torch.cpp

VQ_OK = 0
STATUS_NAMES = {0: "VQ_OK", 1: "VQ_ERR_NULL", 2: "VQ_ERR_SHAPE", 3: "VQ_ERR_ALIGN",
                4: "VQ_ERR_WORKSPACE", 5: "VQ_ERR_LAUNCH", 6: "VQ_ERR_ARCH", 7: "VQ_ERR_BITS"}

# name -> (restype, argtypes); mirrors include/vq.h
_P, _I, _SZ = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
SIGNATURES = {
    "vq_quantize_per_token": (_I, [_P, _P, _P, _P, _I, _I, _P]),
    "vq_gelu_quantize": (_I, [_P, _I, _P, _P, _P, _I, _I, _P]),
    "vq_layernorm_quantize": (_I, [_P, _P, _P, _I, ctypes.c_float, _P, _P, _P, _I, _I, _P]),
    "vq_residual_quantize": (_I, [_P, _P, _P, _I, _P, _P, _P, _P, _I, _I, _P]),
    "vq_channel_absmax": (_I, [_P, _I, _P, _I, _I, _I, _P]),
    "vq_balance_mask": (_I, [_P, _P, ctypes.c_float, _P, _P, _I, _P]),
    "vq_hadamard_quantize": (_I, [_P, _P, _P, _P, _I, _I, _P]),
    "vq_rotate_weight": (_I, [_P, _P, _P, _I, _I, _P]),
    "vq_gemm_f16": (_I, [_P, _P, _P, _P, _I, _I, _I, _P]),
    "vq_quantize_static": (_I, [_P, _P, ctypes.c_float, _P, _I, _I, _P]),
    "vq_gemm_w8a8": (_I, [_P, _P, _P, _P, _P, _P, _P, _I, _I, _I, _P]),
    "vq_gemm_w4a8": (_I, [_P, _P, _P, _P, _P, _P, _P, _I, _I, _I, _P]),
    "vq_linear": (_I, [_P, _P, _P, _I, _P, _P, _P, _P, _SZ, _I, _I, _I, _P]),
    "vq_linear_workspace_bytes": (_SZ, [_I, _I, _I, _I]),
    "vq_layernorm_linear": (_I, [_P, _P, _P, _I, ctypes.c_float, _P, _P, _I, _P, _P, _P, _P, _SZ, _I, _I, _I, _P]),
    "vq_gelu_linear": (_I, [_P, _I, _P, _P, _I, _P, _P, _P, _P, _SZ, _I, _I, _I, _P]),
    "vq_residual_linear": (_I, [_P, _P, _P, _I, _P, _P, _P, _I, _P, _P, _P, _P, _SZ, _I, _I, _I, _P]),
    "vq_hadamard_linear": (_I, [_P, _P, _P, _I, _P, _P, _P, _P, _SZ, _I, _I, _I, _P]),
    "vq_linear_static": (_I, [_P, _P, _P, _I, _P, _P, _P, _I, _I, _I, _P]),
    "vq_quantize_weight": (_I, [_P, _P, _I, _P, _P, _I, _I, _P]),
    "vq_status_string": (ctypes.c_char_p, [_I]),
}


class VqError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {STATUS_NAMES.get(status, status)} ({status_string(status)})")


_lib = None


def lib() -> ctypes.CDLL:
    """Loads libvidiq.so; raises if it has not been built (python -m paper_2406_02540_amd.build)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                f"{LIB_PATH} not found: build it with `python -m paper_2406_02540_amd.build`")
        handle = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in SIGNATURES.items():
            fn = getattr(handle, name)
            fn.restype = res
            fn.argtypes = args
        _lib = handle
    return _lib


def status_string(status: int) -> str:
    return lib().vq_status_string(int(status)).decode()


# order of the entry points' addresses in csrc/vq_torch.cpp
_BOUND = ("vq_quantize_per_token", "vq_gelu_quantize", "vq_layernorm_quantize", "vq_residual_quantize",
          "vq_hadamard_quantize", "vq_quantize_static", "vq_channel_absmax", "vq_balance_mask", "vq_rotate_weight",
          "vq_quantize_weight", "vq_gemm_f16", "vq_gemm_w8a8", "vq_gemm_w4a8", "vq_linear_workspace_bytes", "vq_linear",
          "vq_linear_static", "vq_layernorm_linear", "vq_gelu_linear", "vq_residual_linear", "vq_hadamard_linear")

_ext = None


def _load():
    """Loads the extension and hands it the entry points of libvidiq.so."""
    global _ext
    handle = lib()
    if not os.path.exists(EXT_PATH):
        raise RuntimeError(f"{EXT_PATH} not found: build it with `python -m paper_2406_02540_amd.build`")
    loader = importlib.machinery.ExtensionFileLoader("_vq_torch", EXT_PATH)
    spec = importlib.util.spec_from_file_location("_vq_torch", EXT_PATH, loader=loader)
    rebuild = "build it again with `python -m paper_2406_02540_amd.build`"
    try:
        ext = importlib.util.module_from_spec(spec)
        loader.exec_module(ext)
    except ImportError as e:  # (symbols of another torch)
        raise RuntimeError(f"{EXT_PATH} does not load: {rebuild}") from e
    # the extension holds the layout of the torch that it was compiled against
    if ext.TORCH_VERSION != re.match(r"[\d.]*\d", torch.__version__).group():
        raise RuntimeError(f"{EXT_PATH} was built for torch {ext.TORCH_VERSION}, this is {torch.__version__}: {rebuild}")
    ext.bind(VqError, tuple(ctypes.cast(getattr(handle, n), ctypes.c_void_p).value for n in _BOUND))
    _ext = ext
    return ext


def vq_quantize_per_token(x, chan_mul=None, xq=None, x_scale=None, stream=None):
    """x fp16 [M,K] (+ chan_mul fp32 [K]) -> (xq int8 [M,K], x_scale fp32 [M])."""
    return (_ext or _load()).quantize_per_token(x, chan_mul, xq, x_scale, stream)


def vq_gelu_quantize(h, approximate=False, chan_mul=None, xq=None, x_scale=None, stream=None):
    """GELU (exact or tanh form) fused with the quantizer: h fp16 [M,K] -> (xq, x_scale)."""
    return (_ext or _load()).gelu_quantize(h, approximate, chan_mul, xq, x_scale, stream)


def vq_layernorm_quantize(x, mod_scale=None, mod_shift=None, tokens_per_sample=None, eps=1e-6,
                          chan_mul=None, xq=None, x_scale=None, stream=None):
    """LayerNorm + (1 + scale) y + shift fused with the quantizer: x fp16 [M,K] -> (xq, x_scale)."""
    return (_ext or _load()).layernorm_quantize(x, mod_scale, mod_shift, tokens_per_sample, eps, chan_mul, xq, x_scale,
                                                stream)


def vq_residual_quantize(x, y, gate=None, tokens_per_sample=None, r=None, chan_mul=None, xq=None,
                         x_scale=None, stream=None):
    """r = x + gate * y fused with the quantizer: fp16 [M,K] twice -> (r fp16, xq, x_scale)."""
    return (_ext or _load()).residual_quantize(x, y, gate, tokens_per_sample, r, chan_mul, xq, x_scale, stream)


def vq_channel_absmax(a, amax=None, accumulate=False, stream=None):
    """Per-column absmax of fp16 activations [M,K] or fp32 weights [N,K] -> amax fp32 [K]."""
    return (_ext or _load()).channel_absmax(a, amax, accumulate, stream)


def vq_balance_mask(amax_x, amax_w, alpha, stream=None):
    """Eq. 3: (s, chan_mul = 1/s), fp32 [K] each, from the two absmax statistics."""
    return (_ext or _load()).balance_mask(amax_x, amax_w, alpha, stream)


def vq_hadamard_quantize(x, chan_mul=None, xq=None, x_scale=None, stream=None):
    """Scaling, block Hadamard rotation, per-token quantizer: x fp16 [M,K] -> (xq, x_scale)."""
    return (_ext or _load()).hadamard_quantize(x, chan_mul, xq, x_scale, stream)


def vq_rotate_weight(w, chan_s=None, out=None, stream=None):
    """Weight side of the rotation: w fp32 [N,K] (* chan_s) -> fp32 [N,K]."""
    return (_ext or _load()).rotate_weight(w, chan_s, out, stream)


def vq_gemm_f16(x, w, bias=None, y=None, stream=None):
    """FP16 comparison layer: x fp16 [M,K], w fp16 [N,K] (+ bias fp16 [N]) -> y fp16 [M,N]."""
    return (_ext or _load()).gemm_f16(x, w, bias, y, stream)


def vq_quantize_static(x, scale, chan_mul=None, xq=None, stream=None):
    """One fixed scale for the whole tensor: x fp16 [M,K] -> xq int8 [M,K] (clipped at +-127)."""
    return (_ext or _load()).quantize_static(x, scale, chan_mul, xq, stream)


def vq_gemm_w8a8(xq, x_scale, wq, w_scale, bias=None, y=None, return_acc=False, stream=None):
    """int8 [M,K] x int8 [N,K] -> fp16 [M,N] (and the int32 sums if return_acc)."""
    return (_ext or _load()).gemm_w8a8(xq, x_scale, wq, w_scale, bias, y, return_acc, stream)


def vq_gemm_w4a8(xq, x_scale, wq4, w_scale, bias=None, y=None, return_acc=False, stream=None):
    """int8 [M,K] x packed 4-bit [N,K/2] -> fp16 [M,N] (and the int32 sums if return_acc)."""
    return (_ext or _load()).gemm_w4a8(xq, x_scale, wq4, w_scale, bias, y, return_acc, stream)


def vq_linear_workspace_bytes(M, N, K, w_bits) -> int:
    return int(lib().vq_linear_workspace_bytes(int(M), int(N), int(K), int(w_bits)))


LINEAR_STATIC_SCRATCH_BYTES = 40 << 20  # VQ_LINEAR_STATIC_SCRATCH_BYTES of include/vq.h


def vq_linear_static(x, chan_mul, w, w_bits, w_scale, bias=None, y=None, stream=None):
    """The whole layer with the library's built-in scratch instead of a workspace (the call allocates nothing
    when y is given); layers whose int8 activations exceed LINEAR_STATIC_SCRATCH_BYTES raise VQ_ERR_WORKSPACE."""
    return (_ext or _load()).linear_static(x, chan_mul, w, w_bits, w_scale, bias, y, stream)


def vq_linear(x, chan_mul, w, w_bits, w_scale, bias=None, y=None, workspace=None, stream=None):
    """The whole layer on fp16 activations; workspace is a uint8 device tensor (allocated if None)."""
    return (_ext or _load()).linear(x, chan_mul, w, w_bits, w_scale, bias, y, workspace, stream)


def vq_layernorm_linear(x, w, w_bits, w_scale, mod_scale=None, mod_shift=None, tokens_per_sample=None, eps=1e-6,
                        chan_mul=None, bias=None, y=None, workspace=None, stream=None):
    """LayerNorm + modulation, quantizer and GEMM in one call: x fp16 [M,K] -> y fp16 [M,N]."""
    return (_ext or _load()).layernorm_linear(x, w, w_bits, w_scale, mod_scale, mod_shift, tokens_per_sample, eps,
                                              chan_mul, bias, y, workspace, stream)


def vq_gelu_linear(h, w, w_bits, w_scale, approximate=False, chan_mul=None, bias=None, y=None, workspace=None,
                   stream=None):
    """GELU, quantizer and GEMM in one call: h fp16 [M,K] -> y fp16 [M,N]."""
    return (_ext or _load()).gelu_linear(h, w, w_bits, w_scale, approximate, chan_mul, bias, y, workspace, stream)


def vq_residual_linear(x, y_in, w, w_bits, w_scale, gate=None, tokens_per_sample=None, r=None, chan_mul=None,
                       bias=None, y=None, workspace=None, stream=None):
    """r = x + gate * y_in, quantizer and GEMM in one call: fp16 [M,K] twice -> (r fp16 [M,K], y fp16 [M,N])."""
    return (_ext or _load()).residual_linear(x, y_in, w, w_bits, w_scale, gate, tokens_per_sample, r, chan_mul, bias, y,
                                             workspace, stream)


def vq_hadamard_linear(x, chan_mul, w, w_bits, w_scale, bias=None, y=None, workspace=None, stream=None):
    """Scaling, block Hadamard rotation, quantizer and GEMM in one call (w quantized from rotated weights)."""
    return (_ext or _load()).hadamard_linear(x, chan_mul, w, w_bits, w_scale, bias, y, workspace, stream)


def vq_quantize_weight(w_f32, chan_s=None, w_bits=8, stream=None):
    """W fp32 [N,K] (+ s fp32 [K]) -> (wq int8 [N,K] or packed uint8 [N,K/2], w_scale fp32 [N])."""
    return (_ext or _load()).quantize_weight(w_f32, chan_s, w_bits, stream)

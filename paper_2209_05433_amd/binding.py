"""Binding of libfp8mm.so: same names as the C ABI (include/fp8mm.h), argument marshalling only.
Tensors are torch tensors used as device buffers; every computation happens in the HIP kernels.
The entry points that take tensors come from the extension module _native, the others go through
ctypes, which also gives the raw C ABI (lib()).  There is no fallback: a missing library is an error."""
from __future__ import annotations

import ctypes
import os
import sys

import torch

FP8_E4M3, FP8_E5M2 = 0, 1
FP8_F32, FP8_BF16 = 0, 1
FP8_OK, FP8_ERR_INVALID_ARG, FP8_ERR_UNSUPPORTED, FP8_ERR_DEVICE = 0, 1, 2, 3
FP8_QUANT_NOSAT = 1
FP8_AMAX_WORKSPACE_BYTES = 16384
FP8_SPLITK_STATIC_BYTES = 64 << 20
FP8_GEMM_MFMA8 = 1
FP8_OUT_F32, FP8_OUT_BF16, FP8_OUT_E4M3, FP8_OUT_E5M2 = 0, 1, 2, 3
FP8_PLAN_NO_GEMM, FP8_PLAN_FMA_KERNEL, FP8_PLAN_TILED_256x256, FP8_PLAN_TILED_256x128, FP8_PLAN_MFMA_ANY, FP8_PLAN_TILED_MIXED = 0, 1, 2, 3, 4, 5
FP8_PLAN_ELEMENTWISE_STORES = 16
FP8_MULTI_MAX = 4
FP8_PLAN_PERSISTENT = 32
(FP8_FORM_NO_GEMM, FP8_FORM_FMA, FP8_FORM_TILED_256, FP8_FORM_TILED_192, FP8_FORM_TILED_128, FP8_FORM_TILED_128_PERSISTENT, FP8_FORM_TILED_256_128,
 FP8_FORM_TILED_192_128, FP8_FORM_ANY_256, FP8_FORM_ANY_128, FP8_FORM_SMALL_32x32, FP8_FORM_SMALL_32x64, FP8_FORM_SMALL_64x64,
 FP8_FORM_SMALL_64x64_LINES8, FP8_FORM_SMALL_64x64_LINES4) = range(15)
FP8_KNOB_CAST_PATH, FP8_KNOB_TILE_N, FP8_KNOB_GROUP_M, FP8_KNOB_GEMM_KERNEL, FP8_KNOB_SPLIT_K, FP8_KNOB_CAST_RUN, FP8_KNOB_PERSIST, FP8_KNOB_MIXED, FP8_KNOB_SMALL, FP8_KNOB_PATIENCE, FP8_KNOB_TILE_192, FP8_KNOB_SMALL_64 = range(12)

LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libfp8mm.so")
NATIVE_PATH = os.path.join(os.path.dirname(LIB_PATH), "_native.so")

EXPORTS = (
    "fp8_amax", "fp8_amax_scale", "fp8_amax_scale_multi", "fp8_quantize_multi", "fp8_scale_from_amax_host", "fp8_scale_from_amax", "fp8_quantize",
    "fp8_quantize_dscale", "fp8_quantize_ex", "fp8_dequantize", "fp8_quantize_amax", "fp8_quantize_sr",
    "fp8_scale_from_amax_history", "fp8_scale_from_amax_n", "fp8_amax_rows", "fp8_quantize_rows",
    "fp8_quantize_transpose", "fp8_gemm", "fp8_gemm_dscale", "fp8_gemm_mfma8",
    "fp8_gemm_mfma8_dscale", "fp8_gemm_ex", "fp8_gemm_splitk", "fp8_gemm_splitk_workspace_size", "fp8_gemm_splitk_static", "fp8_gemm_fused", "fp8_scaled_gemm", "fp8_gemm_plan", "fp8_gemm_form", "fp8_set_knob", "fp8_get_knob",
    "fp8_last_error", "fp8_version",
)

_lib = None


class Fp8Error(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__("fp8mm status %d: %s" % (status, message))
        self.status = status


def lib() -> ctypes.CDLL:
    """Loads the built library (build it first: python -m paper_2209_05433_amd.build)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise FileNotFoundError(
            "%s is missing: build the HIP library with __graft_entry__.build() or "
            "`python paper_2209_05433_amd/build.py`; there is no CPU fallback" % LIB_PATH)
    L = ctypes.CDLL(LIB_PATH)
    c = ctypes
    vp, sz, i, i64, f = c.c_void_p, c.c_size_t, c.c_int, c.c_int64, c.c_float
    L.fp8_amax.argtypes, L.fp8_amax.restype = [vp, sz, i, vp, vp], i
    L.fp8_amax_scale.argtypes, L.fp8_amax_scale.restype = [vp, sz, i, i, vp, vp, vp, vp], i
    L.fp8_amax_scale_multi.argtypes, L.fp8_amax_scale_multi.restype = [i, vp, vp, i, vp, vp, vp, vp, vp], i
    L.fp8_quantize_multi.argtypes, L.fp8_quantize_multi.restype = [i, vp, vp, i, vp, vp, vp, vp], i
    L.fp8_scale_from_amax_host.argtypes, L.fp8_scale_from_amax_host.restype = [f, i], f
    L.fp8_scale_from_amax.argtypes, L.fp8_scale_from_amax.restype = [vp, i, vp, vp], i
    L.fp8_quantize.argtypes, L.fp8_quantize.restype = [vp, sz, i, i, f, vp, vp], i
    L.fp8_quantize_dscale.argtypes, L.fp8_quantize_dscale.restype = [vp, sz, i, i, vp, vp, vp], i
    L.fp8_quantize_ex.argtypes, L.fp8_quantize_ex.restype = [vp, sz, i, i, f, vp, i, vp, vp], i
    L.fp8_dequantize.argtypes, L.fp8_dequantize.restype = [vp, sz, i, f, vp, i, vp, vp], i
    L.fp8_gemm.argtypes, L.fp8_gemm.restype = [vp, i, f, vp, i, f, vp, i64, i64, i64, i, vp], i
    L.fp8_gemm_dscale.argtypes, L.fp8_gemm_dscale.restype = [vp, i, vp, vp, i, vp, vp, i64, i64, i64, i, vp], i
    L.fp8_gemm_mfma8.argtypes, L.fp8_gemm_mfma8.restype = L.fp8_gemm.argtypes, i
    L.fp8_gemm_mfma8_dscale.argtypes, L.fp8_gemm_mfma8_dscale.restype = L.fp8_gemm_dscale.argtypes, i
    L.fp8_gemm_ex.argtypes, L.fp8_gemm_ex.restype = [vp, i, i, vp, i, i, vp, i64, i64, i64, i, f, f, vp, vp, i, vp], i
    L.fp8_scaled_gemm.argtypes, L.fp8_scaled_gemm.restype = [vp, vp, i, i, i, i64, i64, i64, i, i, vp, vp, vp, vp, vp, vp, i, i, vp], i
    L.fp8_gemm_splitk.argtypes, L.fp8_gemm_splitk.restype = [vp, i, i, vp, i, i, vp, i64, i64, i64, i, f, f, vp, vp, i, i, vp, sz, vp], i
    L.fp8_gemm_splitk_static.argtypes, L.fp8_gemm_splitk_static.restype = [vp, i, i, vp, i, i, vp, i64, i64, i64, i, f, f, vp, vp, i, i, vp], i
    L.fp8_gemm_splitk_workspace_size.argtypes, L.fp8_gemm_splitk_workspace_size.restype = [i64, i64, i64, i, i, i], sz
    L.fp8_gemm_fused.argtypes, L.fp8_gemm_fused.restype = [vp, i, i, vp, i, i, vp, i, i64, i64, i64, vp, i64, vp, i64, vp, vp, i, vp], i
    L.fp8_quantize_sr.argtypes, L.fp8_quantize_sr.restype = [vp, sz, i, i, f, vp, c.c_uint64, vp, vp], i
    L.fp8_quantize_amax.argtypes, L.fp8_quantize_amax.restype = [vp, sz, i, i, vp, vp, vp, vp], i
    L.fp8_scale_from_amax_history.argtypes, L.fp8_scale_from_amax_history.restype = [vp, sz, i, vp, vp], i
    L.fp8_scale_from_amax_n.argtypes, L.fp8_scale_from_amax_n.restype = [vp, sz, i, vp, vp], i
    L.fp8_amax_rows.argtypes, L.fp8_amax_rows.restype = [vp, i64, i64, i, vp, vp], i
    L.fp8_quantize_rows.argtypes, L.fp8_quantize_rows.restype = [vp, i64, i64, i, i, vp, vp, vp], i
    L.fp8_quantize_transpose.argtypes, L.fp8_quantize_transpose.restype = [vp, i64, i64, i, i, vp, vp, vp, vp], i
    L.fp8_gemm_plan.argtypes, L.fp8_gemm_plan.restype = [vp, i, vp, i, vp, i64, i64, i64, vp], i
    L.fp8_gemm_form.argtypes, L.fp8_gemm_form.restype = [vp, i, vp, i, vp, i64, i64, i64, i, vp, i], i
    L.fp8_set_knob.argtypes, L.fp8_set_knob.restype = [i, i], i
    L.fp8_get_knob.argtypes, L.fp8_get_knob.restype = [i], i
    L.fp8_last_error.argtypes, L.fp8_last_error.restype = [], c.c_char_p
    L.fp8_version.argtypes, L.fp8_version.restype = [], c.c_char_p
    _lib = L
    return L


def dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return FP8_F32
    if t.dtype == torch.bfloat16:
        return FP8_BF16
    raise TypeError("expected a float32 or bfloat16 tensor, got %s" % t.dtype)


def fp8_last_error() -> str:
    return lib().fp8_last_error().decode()


def fp8_version() -> str:
    return lib().fp8_version().decode()


def fp8_set_knob(knob: int, value: int) -> int:
    """Sets a tuning knob (fp8_knob_t) and returns its previous value."""
    old = lib().fp8_set_knob(int(knob), int(value))
    if old < 0:
        raise Fp8Error(-old, lib().fp8_last_error().decode())
    return old


def fp8_get_knob(knob: int) -> int:
    v = lib().fp8_get_knob(int(knob))
    if v < 0:
        raise Fp8Error(-v, lib().fp8_last_error().decode())
    return v


def fp8_gemm_plan(A: torch.Tensor, transA: bool, B: torch.Tensor, transB: bool, C: torch.Tensor, sB_per_column=None) -> int:
    """Which kernel the GEMM entry points would run for these tensors, the kernel of small tiles apart (an
    fp8_plan_t, possibly ORed with FP8_PLAN_ELEMENTWISE_STORES and FP8_PLAN_PERSISTENT); nothing is launched."""
    M, K = (A.shape[1], A.shape[0]) if transA else A.shape
    N = B.shape[0] if transB else B.shape[1]
    plan = lib().fp8_gemm_plan(A.data_ptr(), int(bool(transA)), B.data_ptr(), int(bool(transB)), C.data_ptr(), M, N, K,
                               None if sB_per_column is None else sB_per_column.data_ptr())
    if plan < 0:
        raise Fp8Error(-plan, lib().fp8_last_error().decode())
    return plan


def fp8_gemm_form(A: torch.Tensor, transA: bool, B: torch.Tensor, transB: bool, C: torch.Tensor, out_kind: int, sB_per_column=None, flags: int = 0) -> int:
    """The form of the kernel (an fp8_form_t) that a product of these tensors runs, small tiles and 256 x 192 tiles included."""
    M, K = (A.shape[1], A.shape[0]) if transA else A.shape
    N = B.shape[0] if transB else B.shape[1]
    form = lib().fp8_gemm_form(A.data_ptr(), int(bool(transA)), B.data_ptr(), int(bool(transB)), C.data_ptr(), M, N, K, int(out_kind),
                               None if sB_per_column is None else sB_per_column.data_ptr(), int(flags))
    if form < 0:
        raise Fp8Error(-form, lib().fp8_last_error().decode())
    return form


def fp8_scale_from_amax_host(amax: float, fmt: int) -> float:
    return float(lib().fp8_scale_from_amax_host(float(amax), fmt))


def fp8_gemm_splitk_workspace_size(M: int, N: int, K: int, transA: bool, transB: bool, splits: int = 0) -> int:
    return int(lib().fp8_gemm_splitk_workspace_size(M, N, K, int(bool(transA)), int(bool(transB)), int(splits)))


# The entry points that take tensors: unpacked in C (csrc/native_binding.cpp; their argument names and
# defaults are in the docstrings there), since marshalling them here costs more than a short launch.
TENSOR_CALLS = (
    "fp8_amax", "fp8_amax_scale", "fp8_amax_scale_multi", "fp8_quantize_multi", "fp8_scale_from_amax", "fp8_quantize", "fp8_quantize_dscale",
    "fp8_quantize_ex", "fp8_dequantize", "fp8_quantize_amax", "fp8_quantize_sr", "fp8_scale_from_amax_history", "fp8_scale_from_amax_n",
    "fp8_amax_rows", "fp8_quantize_rows", "fp8_quantize_transpose", "fp8_gemm", "fp8_gemm_dscale", "fp8_gemm_mfma8", "fp8_gemm_mfma8_dscale",
    "fp8_gemm_ex", "fp8_gemm_splitk", "fp8_gemm_splitk_static", "fp8_gemm_fused", "fp8_scaled_gemm",
)

_native = None


def native():
    """The built binding module (build it first, with the library); its absence is an error."""
    global _native
    if _native is None:
        lib()
        if not os.path.exists(NATIVE_PATH):
            raise FileNotFoundError("%s is missing: build it with __graft_entry__.build() or `python paper_2209_05433_amd/build.py`" % NATIVE_PATH)
        from importlib.machinery import ExtensionFileLoader
        from importlib.util import module_from_spec, spec_from_loader
        name = __package__ + "._native"
        m = module_from_spec(spec_from_loader(name, ExtensionFileLoader(name, NATIVE_PATH)))
        m.__spec__.loader.exec_module(m)
        m.set_error(Fp8Error)
        sys.modules[name] = _native = m              # (under the name that its functions are pickled by)
    return _native


def __getattr__(name):
    """Loads the binding at the first use of an entry point, not at import (the build imports this package)."""
    if name not in TENSOR_CALLS:
        raise AttributeError("module %r has no attribute %r" % (__name__, name))
    globals()[name] = fn = getattr(native(), name)
    return fn

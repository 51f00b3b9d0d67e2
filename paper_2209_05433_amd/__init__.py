"""MI355X-native scaled-FP8 matrix multiply path (amax -> scale -> cast -> FP8 GEMM ->
unscale) of arXiv 2209.05433, as hand-written HIP kernels behind a C ABI.

The functions re-exported here have the names and argument order of include/fp8mm.h and
only marshal arguments; the library is loaded on first use and its absence is an error.
"""
import os

from . import binding
from .binding import (  # noqa: F401
    FP8_E4M3, FP8_E5M2, FP8_F32, FP8_BF16,
    FP8_OK, FP8_ERR_INVALID_ARG, FP8_ERR_UNSUPPORTED, FP8_ERR_DEVICE,
    EXPORTS, LIB_PATH, Fp8Error, lib,
    FP8_MULTI_MAX, FP8_AMAX_WORKSPACE_BYTES, fp8_scale_from_amax_host, FP8_QUANT_NOSAT,
    fp8_gemm_splitk_workspace_size, FP8_SPLITK_STATIC_BYTES, FP8_GEMM_MFMA8,
    FP8_OUT_F32, FP8_OUT_BF16, FP8_OUT_E4M3, FP8_OUT_E5M2, fp8_gemm_plan,
    FP8_PLAN_NO_GEMM, FP8_PLAN_FMA_KERNEL, FP8_PLAN_TILED_256x256, FP8_PLAN_TILED_256x128, FP8_PLAN_MFMA_ANY, FP8_PLAN_TILED_MIXED, FP8_PLAN_ELEMENTWISE_STORES,
    fp8_set_knob, fp8_get_knob, FP8_KNOB_CAST_PATH, FP8_KNOB_TILE_N, FP8_KNOB_GROUP_M, FP8_KNOB_GEMM_KERNEL, FP8_KNOB_SPLIT_K, FP8_KNOB_CAST_RUN, FP8_KNOB_PERSIST, FP8_KNOB_MIXED, FP8_KNOB_SMALL, FP8_KNOB_PATIENCE, FP8_KNOB_TILE_192, FP8_KNOB_SMALL_64, FP8_PLAN_PERSISTENT,
    fp8_gemm_form, FP8_FORM_NO_GEMM, FP8_FORM_FMA, FP8_FORM_TILED_256, FP8_FORM_TILED_192, FP8_FORM_TILED_128, FP8_FORM_TILED_128_PERSISTENT,
    FP8_FORM_TILED_256_128, FP8_FORM_TILED_192_128, FP8_FORM_ANY_256, FP8_FORM_ANY_128, FP8_FORM_SMALL_32x32, FP8_FORM_SMALL_32x64,
    FP8_FORM_SMALL_64x64, FP8_FORM_SMALL_64x64_LINES8, FP8_FORM_SMALL_64x64_LINES4,
    fp8_last_error, fp8_version,
)

# What `import *` brings: the names above and the entry points that take tensors (looked up only where they are built).
__all__ = [n for n in globals() if not n.startswith("_") and n != "os"]
if os.path.exists(binding.NATIVE_PATH):
    __all__ += binding.TENSOR_CALLS


def __getattr__(name):
    """The entry points that take tensors: bound when first asked for, the library is loaded then."""
    if name not in binding.TENSOR_CALLS:
        raise AttributeError("module %r has no attribute %r" % (__name__, name))
    globals()[name] = fn = getattr(binding, name)
    return fn

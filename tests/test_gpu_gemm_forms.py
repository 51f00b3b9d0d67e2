"""Every form of the matrix-core kernels through the products that the dispatcher would send to one of
them: each form is pinned by knobs, so that a later change of the dispatcher's rules leaves it covered.
The checks are those of the tests that run at default knobs (test_gpu_gemm, test_gpu_gemm_fused,
test_gpu_ragged), against the oracle."""
import contextlib

import numpy as np
import pytest
import torch

import paper_2209_05433_amd as fp8
import test_gpu_gemm as gemm
import test_gpu_gemm_fused as fused
import test_gpu_ragged as ragged
from gpu_util import knob

pytestmark = pytest.mark.gpu

TILE_N, KERNEL, SMALL = fp8.FP8_KNOB_TILE_N, fp8.FP8_KNOB_GEMM_KERNEL, fp8.FP8_KNOB_SMALL
SMALL_FORMS = {"32x32": {SMALL: 2}, "32x64": {SMALL: 3}, "64x64": {SMALL: 4}}
# (a problem that the tiled kernel does not take runs on the any-shape form of the same width)
FORMS = {"tiled 256": {TILE_N: 256}, "tiled 128": {TILE_N: 128}, "any 256": {KERNEL: 2, TILE_N: 256}, "any 128": {KERNEL: 2, TILE_N: 128}, **SMALL_FORMS}


@contextlib.contextmanager
def pinned(knobs):
    with contextlib.ExitStack() as stack:
        for which, value in knobs.items():
            stack.enter_context(knob(which, value))
        yield


# Beside the sizes of the default test: several trips of every wave along K and a remainder, and a
# row-contiguous operand whose rows are shorter than a vector
EDGES = ragged.SMALL + [(9, 70, 5000, 0), (130, 12, 4133, 3), (12, 200, 4133, 2), (200, 330, 6200, 1), (64, 64, 256, 1)]


@pytest.mark.parametrize("form", sorted(SMALL_FORMS))
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,off", EDGES)
def test_small_forms_at_their_edges(M, N, K, off, transA, transB, form):
    with pinned(SMALL_FORMS[form]):
        ragged.test_small_tiles_at_their_edges(M, N, K, off, transA, transB)


# 64 x 64 tiles of operands that are both contiguous along K have three forms: chunks of 64 and of 128 in four waves, of 128 in eight
FORMS_64 = {1: fp8.FP8_FORM_SMALL_64x64, 2: fp8.FP8_FORM_SMALL_64x64_LINES8, 3: fp8.FP8_FORM_SMALL_64x64_LINES4}


@pytest.mark.parametrize("which", sorted(FORMS_64))
@pytest.mark.parametrize("M,N,K,off", EDGES + [(1030, 1100, 2601, 1), (1088, 1024, 2560, 0), (1500, 1505, 200, 0), (1500, 1505, 67, 2), (61, 190, 1281, 0), (64, 128, 2048, 0)])
def test_64x64_forms_of_k_contiguous_operands(M, N, K, off, which):
    with pinned({**SMALL_FORMS["64x64"], fp8.FP8_KNOB_SMALL_64: which}):
        assert fp8.lib().fp8_gemm_form(1 << 20, 0, 1 << 24, 1, 1 << 28, M, N, K, fp8.FP8_OUT_F32, None, 0) == FORMS_64[which]
        ragged.test_small_tiles_at_their_edges(M, N, K, off, 0, 1)


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("mode", fused.MODES)
def test_outputs_of_every_form(mode, form):
    """Special values and output maxima with NaN, FP8 outputs below and beyond the format's maximum, factors per
    row and column, sums that are exact."""
    with pinned(FORMS[form]):
        fused.test_fp8_output_special_values_and_amax_nan(mode)
        for kind in (fp8.FP8_OUT_E4M3, fp8.FP8_OUT_E5M2):
            fused.test_fp8_output_with_output_scale_and_amax(kind, mode)
            fused.test_fp8_output_is_the_oracle_byte_where_sums_are_exact(kind, mode)
        for a_vec in (0, 1):
            for b_vec in (0, 1):
                fused.test_per_channel_scales(a_vec, b_vec, mode)
        gemm.test_one_hot_probes_over_a_multi_tile_problem(mode)
        gemm.test_non_finite_operands_keep_their_class(mode)
        for fmtA, fmtB in gemm.MIXES:
            gemm.test_random_codes_all_format_mixes(fmtA, fmtB, fp8.FP8_F32, mode)
    if mode == "f16":
        with pinned(FORMS[form]):
            fused.test_per_channel_scales_are_not_swapped_or_shifted()


@pytest.mark.parametrize("form", ["any 128", "any 256", *sorted(SMALL_FORMS)])
def test_factors_per_column_are_rounded_once(form):
    """Off the tiled kernel an output is acc * fl32(1 / (sA sB)), the reciprocal formed in 64 bits and rounded once: the
    bits of that expression where the sums are exact, and a finite product of factors whose own reciprocals leave the
    32-bit range (1 / 1e-39 = inf, 1 / (1e-39 * 1e5) = 1e34)."""
    rng = np.random.default_rng(71)
    M, N, K = 300, 333, 530                      # (rows of B and of the output start at odd places: not the tiled kernel's)
    A, B = fused.int_codes(rng, (M, K)), fused.int_codes(rng, (K, N))
    S = fused.oracle.gemm_rows(A, fused.E4M3, B, fused.E4M3)[0].astype(np.float32)
    sB = rng.uniform(0.5, 4.0, N).astype(np.float32)
    with pinned(FORMS[form]):
        for sA, col in ((rng.uniform(0.5, 4.0, M).astype(np.float32), sB), (np.float32(1.7), sB), (np.full(M, 1e-39, np.float32), sB * np.float32(1e5))):
            a = np.broadcast_to(np.asarray(sA, np.float64), (M,))[:, None]
            want = S * (1.0 / (a * col.astype(np.float64))).astype(np.float32)
            assert np.all(np.isfinite(want))
            got = fused.run_fused(A, fused.E4M3, B, fused.E4M3, fp8.FP8_OUT_F32, sA, col)[0].cpu().numpy()
            assert np.array_equal(got, want), "%d of %d outputs differ" % (np.count_nonzero(got != want), want.size)


# K of one row, of less than a stage, one less and one more than a pair of stages, several pairs and a remainder
@pytest.mark.parametrize("K", [1, 63, 127, 129, 1000, 2305])
@pytest.mark.parametrize("knobs", [{TILE_N: 256}, {TILE_N: 128}, {fp8.FP8_KNOB_TILE_192: 2}, {fp8.FP8_KNOB_TILE_192: 2, fp8.FP8_KNOB_MIXED: 2}],
                         ids=["256", "128", "192", "192 and 128"])
def test_tiled_kernel_over_any_k_of_operands_contiguous_along_m_and_n(knobs, K):
    """Sums of integers, exact; guard bytes of NaN behind the operands and around the output."""
    rng = np.random.default_rng(K)
    M, N = 272, 592
    for fmtA, fmtB, flags in ((fused.E4M3, fused.E4M3, 0), (fused.E5M2, fused.E4M3, fp8.FP8_GEMM_MFMA8)):
        A = fused.oracle.quantize(rng.integers(-3, 4, (M, K)).astype(np.float32), fmtA, 1.0)
        B = fused.oracle.quantize(rng.integers(-3, 4, (K, N)).astype(np.float32), fmtB, 1.0)
        want = fused.oracle.gemm_rows(A, fmtA, B, fmtB)[0]
        dA, dB = (torch.full((x.size + 512,), 0x7F, dtype=torch.uint8, device="cuda") for x in (A, B))
        dA, dB = dA[:A.size].view(K, M), dB[:B.size].view(K, N)
        dA.copy_(torch.from_numpy(np.ascontiguousarray(A.T)))
        dB.copy_(torch.from_numpy(B))
        buf = torch.full((M * N + 128,), 9.0, device="cuda")
        C = buf[64:64 + M * N].view(M, N)
        with pinned(knobs):
            assert fp8.fp8_gemm_form(dA, True, dB, False, C, fp8.FP8_OUT_F32, None, flags) in (
                fp8.FP8_FORM_TILED_256, fp8.FP8_FORM_TILED_128, fp8.FP8_FORM_TILED_192, fp8.FP8_FORM_TILED_192_128)
            fp8.fp8_gemm_ex(dA, fmtA, True, dB, fmtB, False, C, 1.0, 1.0, flags=flags)
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy().astype(np.float64), want)
        assert bool((buf[:64] == 9).all()) and bool((buf[64 + M * N:] == 9).all())

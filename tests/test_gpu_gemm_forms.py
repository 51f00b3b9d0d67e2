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
from gpu_util import knob, launches

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


# rows in memory of one byte to one less than a vector; K of one row, of rows that together are less than a vector, of several chunks and a remainder
@pytest.mark.parametrize("K", [1, 3, 15, 65, 1000])
@pytest.mark.parametrize("ext", [1, 2, 5, 8, 15])
@pytest.mark.parametrize("tile", [2, 3, 4], ids=["32x32", "32x64", "64x64"])
def test_small_tiles_of_rows_shorter_than_a_vector(tile, ext, K):
    """Operands stored K x M / K x N with M, N < 16: sums of integers, exact; guard bytes of NaN before and behind the operands, which begin anywhere."""
    rng = np.random.default_rng(100 * ext + K)
    for M, N, transA, transB in ((ext, 40, 1, 1), (40, ext, 0, 0), (ext, ext, 1, 0), (ext, 100, 1, 0)):
        A = fused.oracle.quantize(rng.integers(-3, 4, (M, K)).astype(np.float32), fused.E4M3, 1.0)
        B = fused.oracle.quantize(rng.integers(-3, 4, (K, N)).astype(np.float32), fused.E5M2, 1.0)
        want = fused.oracle.gemm_rows(A, fused.E4M3, B, fused.E5M2)[0]
        dev = []
        for x, off in ((A.T if transA else A, 33), (B.T if transB else B, 7)):
            buf = torch.full((x.size + 128,), 0x7F, dtype=torch.uint8, device="cuda")
            t = buf[off:off + x.size].view(x.shape)
            t.copy_(torch.from_numpy(np.ascontiguousarray(x)))
            dev.append(t)
        C = torch.full((M, N), 9.0, device="cuda")
        with pinned({fp8.FP8_KNOB_SMALL: tile}):
            fp8.fp8_gemm_ex(dev[0], fused.E4M3, transA, dev[1], fused.E5M2, transB, C, 1.0, 1.0)
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy().astype(np.float64), want), (M, N, transA, transB)


def test_rows_shorter_than_a_vector_cost_no_more_than_a_vector():
    """A product with 15 columns, stored K x 15, against the same one with 16: 30 us against 18 (byte by byte 112)."""
    a = torch.randint(0, 100, (16384, 4096), dtype=torch.uint8, device="cuda")
    took = []
    for N in (15, 16):
        b, c = torch.randint(0, 100, (4096, N), dtype=torch.uint8, device="cuda"), torch.empty((16384, N), device="cuda")
        best, ev = 1e9, [torch.cuda.Event(True) for _ in range(2)]
        for _ in range(5):
            ev[0].record()
            for _ in range(20):
                fp8.fp8_gemm_ex(a, fused.E4M3, False, b, fused.E4M3, False, c, 1.0, 1.0)
            ev[1].record()
            torch.cuda.synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) * 50.0)
        took.append(best)
    assert took[0] < 3.0 * took[1], took


# one and two chunks of 64, a chunk and one element; rows of A that end inside a vector and rows shorter than one
@pytest.mark.parametrize("K", [7, 64, 65, 128])
@pytest.mark.parametrize("kind", [fp8.FP8_OUT_F32, fp8.FP8_OUT_BF16, fp8.FP8_OUT_E4M3])
@pytest.mark.parametrize("M,transA,transB", [(70, 0, 1), (67, 1, 0), (5, 1, 1)])
def test_64x64_tiles_with_as_many_waves_as_chunks(M, transA, transB, kind, K):
    """Beyond 1024 tiles a workgroup has no waves that K leaves without a chunk: outputs and their maximum bit for bit those of
    the same columns in products of fewer tiles, with factors per row and column."""
    rng = np.random.default_rng(K)
    N, part = 70003, 17500                                # 1094 columns of tiles or more, 274
    A, B = gemm.random_codes(rng, (M, K), fused.E4M3), gemm.random_codes(rng, (N, K), fused.E5M2)
    dA = torch.from_numpy(np.ascontiguousarray(A.T) if transA else A).cuda()
    dB = torch.from_numpy(B).cuda()
    sA, sB, sD = torch.rand(M, device="cuda") + 0.5, torch.rand(N, device="cuda") + 0.5, torch.full((1,), 1e-3, device="cuda")
    out = {fp8.FP8_OUT_F32: torch.float32, fp8.FP8_OUT_BF16: torch.bfloat16}.get(kind, torch.uint8)

    def run(b, factors):
        d, amax = torch.zeros((M, b.shape[0]), dtype=out, device="cuda"), torch.zeros(1, device="cuda")
        with pinned({fp8.FP8_KNOB_SMALL: 4, fp8.FP8_KNOB_SMALL_64: 1}):
            ran = launches(lambda: fp8.fp8_gemm_fused(dA, fused.E4M3, transA, b if transB else b.t().contiguous(), fused.E5M2, transB, d, kind, sA, factors,
                                                      sD if out == torch.uint8 else None, amax))[-1][1]
            fp8.fp8_gemm_fused(dA, fused.E4M3, transA, b if transB else b.t().contiguous(), fused.E5M2, transB, d, kind, sA, factors,
                               sD if out == torch.uint8 else None, amax)
        return d, amax.item(), ran

    whole, amax, threads = run(dB, sB)
    assert threads == (64 if K <= 64 else 128)
    most = 0.0
    for at in range(0, N, part):
        d, m, threads = run(dB[at:at + part].contiguous(), sB[at:at + part].contiguous())
        assert threads == 256
        most = max(most, m)
        assert torch.equal(d.view(torch.uint8), whole[:, at:at + part].contiguous().view(torch.uint8)), at
    assert most == amax

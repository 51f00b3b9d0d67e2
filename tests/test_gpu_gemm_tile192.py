"""The tiled kernel's tile of 256 x 192, alone and with 128-wide tiles behind it in one launch: every storage order, mode
and output kind at the edges of the tile, against the oracle where the sums are exact and bit for bit against the
256-wide tile (every output adds its K in the same order whatever the tile)."""
import contextlib

import numpy as np
import pytest
import torch

import oracle
import paper_2209_05433_amd as fp8
from gpu_util import knob, out_to_f64, to_dev

pytestmark = pytest.mark.gpu

E4M3, E5M2 = fp8.FP8_E4M3, fp8.FP8_E5M2
OUT = {fp8.FP8_OUT_F32: torch.float32, fp8.FP8_OUT_BF16: torch.bfloat16, fp8.FP8_OUT_E4M3: torch.uint8, fp8.FP8_OUT_E5M2: torch.uint8}
FLAGS = {"f16": 0, "mfma8": fp8.FP8_GEMM_MFMA8}
# one whole tile; one column more than a tile and than a half of it; a tile and a wave's half; K of one chunk, of an odd
# number of stages, of a partly filled pair
SHAPES = [(256, 192, 128), (272, 208, 16), (512, 96, 192), (304, 288, 1040), (128, 592, 320), (624, 384, 2096)]


def product(dA, tA, dB, tB, shape, kind, sB, sD, flags, fmts=(E4M3, E5M2), sA=None):
    M, N = shape
    guard = 64
    buf = torch.full((M * N + 2 * guard,), 9, dtype=OUT[kind], device="cuda")
    D = buf[guard:guard + M * N].view(M, N)
    amax = torch.full((1,), -1.0, device="cuda")
    fp8.fp8_gemm_fused(dA, fmts[0], tA, dB, fmts[1], tB, D, kind, torch.full((1,), 2.0, device="cuda") if sA is None else sA, sB, sD, amax, flags)
    torch.cuda.synchronize()
    assert bool((buf[:guard] == 9).all()) and bool((buf[guard + M * N:] == 9).all()), "wrote outside the output"
    return D, amax


# alone, and (where N leaves room) in half of the columns with 128-wide tiles behind
KNOBS = {"alone": {fp8.FP8_KNOB_TILE_192: 2}, "behind": {fp8.FP8_KNOB_TILE_192: 2, fp8.FP8_KNOB_MIXED: 2}}


@contextlib.contextmanager
def knobs(values):
    with contextlib.ExitStack() as stack:
        for which, value in values.items():
            stack.enter_context(knob(which, value))
        yield


@pytest.mark.parametrize("form", sorted(KNOBS))
@pytest.mark.parametrize("mode", sorted(FLAGS))
@pytest.mark.parametrize("fmts", [(E4M3, E4M3), (E4M3, E5M2), (E5M2, E4M3), (E5M2, E5M2)])
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_every_output_kind_at_the_edges_of_the_tile(transA, transB, fmts, mode, form):
    rng = np.random.default_rng(192 + 2 * transA + transB)
    for M, N, K in SHAPES:
        if transB:
            N += 5                                      # (any N goes where B is stored N x K)
        if form == "behind" and N <= 192:
            continue
        ai, bi = rng.integers(-4, 5, (M, K)).astype(np.float32), rng.integers(-4, 5, (K, N)).astype(np.float32)
        want = ai.astype(np.float64) @ bi.astype(np.float64)
        Aq, Bq = oracle.quantize(ai, fmts[0], 1.0), oracle.quantize(bi, fmts[1], 1.0)
        dA = to_dev(np.ascontiguousarray(Aq.T) if transA else Aq)
        dB = to_dev(np.ascontiguousarray(Bq.T) if transB else Bq)
        for kind in OUT:
            for per_row, per_column in ((False, False), (False, True), (True, True)):
                sA = torch.from_numpy(2.0 ** rng.integers(-2, 3, M if per_row else 1)).float().cuda()
                sB = torch.from_numpy(2.0 ** rng.integers(-2, 3, N if per_column else 1)).float().cuda()
                sD = torch.full((1,), 0.25, device="cuda") if kind >= fp8.FP8_OUT_E4M3 else None
                what = (M, N, K, kind, per_row, per_column)
                with knobs(KNOBS[form]):
                    runs = fp8.fp8_gemm_form(dA, transA, dB, transB, dA, kind, None, FLAGS[mode])
                    assert runs == (fp8.FP8_FORM_TILED_192 if form == "alone" else fp8.FP8_FORM_TILED_192_128), what
                    D, amax = product(dA, transA, dB, transB, (M, N), kind, sB, sD, FLAGS[mode], fmts, sA)
                with knob(fp8.FP8_KNOB_TILE_N, 256):
                    D256, amax256 = product(dA, transA, dB, transB, (M, N), kind, sB, sD, FLAGS[mode], fmts, sA)
                assert torch.equal(D, D256) and torch.equal(amax, amax256), what
                ref = want / sA.cpu().numpy().astype(np.float64)[:, None] / sB.cpu().numpy().astype(np.float64)
                assert float(amax) == np.max(np.abs(ref))
                if kind == fp8.FP8_OUT_F32:             # (integers and powers of two: exact)
                    assert np.array_equal(out_to_f64(D), ref), what
                elif kind >= fp8.FP8_OUT_E4M3:
                    fmt = E4M3 if kind == fp8.FP8_OUT_E4M3 else E5M2
                    assert np.array_equal(D.cpu().numpy(), oracle.quantize((ref * 0.25).astype(np.float32), fmt, 1.0)), what


@pytest.mark.parametrize("form", sorted(KNOBS))
@pytest.mark.parametrize("mode", sorted(FLAGS))
@pytest.mark.parametrize("fmts", [(E4M3, E4M3), (E5M2, E4M3)])
def test_nan_and_infinity_stay_in_their_row_and_column(fmts, mode, form):
    """A NaN code in row 130 of A and one in column 200 of B, an infinity (E5M2) in row 7: those rows and that column and the
    output maximum are not finite, as with the 256-wide tile, and every other output is exact."""
    rng = np.random.default_rng(3)
    M, N, K = 272, 400, 208
    ai, bi = rng.integers(1, 5, (M, K)).astype(np.float32), rng.integers(1, 5, (K, N)).astype(np.float32)
    want = ai.astype(np.float64) @ bi.astype(np.float64) / 2.0
    Aq, Bq = oracle.quantize(ai, fmts[0], 1.0), oracle.quantize(bi, fmts[1], 1.0)
    Aq[130, 77], Bq[150, 200] = 0x7F, 0x7F
    if fmts[0] == E5M2:
        Aq[7, 3] = 0x7C
        want[7] = np.inf
    want[130], want[:, 200] = np.nan, np.nan
    one = torch.ones(1, device="cuda")
    for kind in (fp8.FP8_OUT_F32, fp8.FP8_OUT_E4M3):
        sD = torch.full((1,), 0.25, device="cuda") if kind == fp8.FP8_OUT_E4M3 else None
        with knobs(KNOBS[form]):
            D, amax = product(to_dev(Aq), 0, to_dev(Bq), 0, (M, N), kind, one, sD, FLAGS[mode], fmts)
        assert bool(torch.isnan(amax))
        if kind == fp8.FP8_OUT_F32:
            assert np.array_equal(out_to_f64(D), want, equal_nan=True)
        else:
            assert np.array_equal(D.cpu().numpy() & 0x7F, oracle.quantize((want * 0.25).astype(np.float32), E4M3, 1.0) & 0x7F)


# sizes at which the dispatcher takes the tile by itself: two full rounds of it; a single round, where K is short; a round of it and
# 128-wide tiles for the rest of N
TAKEN = {(4096, 6144, 2048): fp8.FP8_FORM_TILED_192, (2816, 4416, 384): fp8.FP8_FORM_TILED_192,
         (1984, 8576, 4112): fp8.FP8_FORM_TILED_192_128, (3296, 6192, 880): fp8.FP8_FORM_TILED_192_128}


@pytest.mark.parametrize("mode", sorted(FLAGS))
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", sorted(TAKEN))
def test_the_dispatchers_choice_gives_the_bits_of_the_other_tiles(M, N, K, transA, transB, mode):
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    # codes up to 2^3 (E4M3) and 2^2 (E5M2) of either sign: sums around zero
    dA, dB = (torch.randint(0, top, s, dtype=torch.uint8, device="cuda", generator=g) | torch.randint(0, 2, s, dtype=torch.uint8, device="cuda", generator=g) << 7
              for top, s in ((0x51, (K, M) if transA else (M, K)), (0x45, (N, K) if transB else (K, N))))
    sB = torch.rand(N, device="cuda", generator=g) + 0.5
    sD = None
    for kind in (fp8.FP8_OUT_F32, fp8.FP8_OUT_BF16, fp8.FP8_OUT_E4M3):
        buf = torch.empty((M, N), dtype=OUT[kind], device="cuda")
        assert fp8.fp8_gemm_form(dA, transA, dB, transB, buf, kind, sB, FLAGS[mode]) == TAKEN[M, N, K]
        factor = sD if kind >= fp8.FP8_OUT_E4M3 else None
        D, amax = product(dA, transA, dB, transB, (M, N), kind, sB, factor, FLAGS[mode])
        with knob(fp8.FP8_KNOB_TILE_192, 1):
            assert fp8.fp8_gemm_form(dA, transA, dB, transB, buf, kind, sB, FLAGS[mode]) not in (fp8.FP8_FORM_TILED_192, fp8.FP8_FORM_TILED_192_128)
            D1, amax1 = product(dA, transA, dB, transB, (M, N), kind, sB, factor, FLAGS[mode])
        assert torch.equal(D, D1) and torch.equal(amax, amax1), (kind, int((D != D1).sum()))
        if kind == fp8.FP8_OUT_F32:
            sD = (100.0 / D.std()).reshape(1)           # the FP8 outputs: 448 is at four and a half deviations
        elif kind == fp8.FP8_OUT_E4M3:
            bytes_, counts = torch.unique(D, return_counts=True)
            assert len(bytes_) > 200 and int(counts.max()) < 0.05 * M * N, "outputs that do not tell a wrong sum from a right one"

"""The tiled kernel's tile of 256 x 192, alone and with 128-wide tiles behind it in one launch: every storage order, mode
and output kind at the edges of the tile, against the oracle where the sums are exact and bit for bit against the
256-wide tile (every output adds its K in the same order whatever the tile)."""
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


def product(dA, tA, dB, tB, shape, kind, sB, sD, flags):
    M, N = shape
    guard = 64
    buf = torch.full((M * N + 2 * guard,), 9, dtype=OUT[kind], device="cuda")
    D = buf[guard:guard + M * N].view(M, N)
    amax = torch.full((1,), -1.0, device="cuda")
    fp8.fp8_gemm_fused(dA, E4M3, tA, dB, E5M2, tB, D, kind, torch.full((1,), 2.0, device="cuda"), sB, sD, amax, flags)
    torch.cuda.synchronize()
    assert bool((buf[:guard] == 9).all()) and bool((buf[guard + M * N:] == 9).all()), "wrote outside the output"
    return D, amax


@pytest.mark.parametrize("mode", sorted(FLAGS))
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_every_output_kind_at_the_edges_of_the_tile(transA, transB, mode):
    rng = np.random.default_rng(192 + 2 * transA + transB)
    for M, N, K in SHAPES:
        if transB:
            N += 5                                      # (any N goes where B is stored N x K)
        ai, bi = rng.integers(-4, 5, (M, K)).astype(np.float32), rng.integers(-4, 5, (K, N)).astype(np.float32)
        want = (ai.astype(np.float64) @ bi.astype(np.float64)) / 2.0
        Aq, Bq = oracle.quantize(ai, E4M3, 1.0), oracle.quantize(bi, E5M2, 1.0)
        dA = to_dev(np.ascontiguousarray(Aq.T) if transA else Aq)
        dB = to_dev(np.ascontiguousarray(Bq.T) if transB else Bq)
        for kind in OUT:
            for per_column in (False, True):
                sB = torch.from_numpy(2.0 ** rng.integers(-2, 3, N if per_column else 1)).float().cuda()
                sD = torch.full((1,), 0.25, device="cuda") if kind >= fp8.FP8_OUT_E4M3 else None
                with knob(fp8.FP8_KNOB_TILE_192, 2):
                    D, amax = product(dA, transA, dB, transB, (M, N), kind, sB, sD, FLAGS[mode])
                with knob(fp8.FP8_KNOB_TILE_N, 256):
                    D256, amax256 = product(dA, transA, dB, transB, (M, N), kind, sB, sD, FLAGS[mode])
                assert torch.equal(D, D256) and torch.equal(amax, amax256), (M, N, K, kind, per_column)
                ref = want / sB.cpu().numpy().astype(np.float64)
                assert float(amax) == np.max(np.abs(ref))
                if kind == fp8.FP8_OUT_F32:             # (integers and powers of two: exact)
                    assert np.array_equal(out_to_f64(D), ref), (M, N, K, per_column)
                elif kind >= fp8.FP8_OUT_E4M3:
                    fmt = E4M3 if kind == fp8.FP8_OUT_E4M3 else E5M2
                    assert np.array_equal(D.cpu().numpy(), oracle.quantize((ref * 0.25).astype(np.float32), fmt, 1.0)), (M, N, K, per_column)


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

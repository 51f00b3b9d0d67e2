"""The binding of the entry points that take tensors: which memory it hands out, which arguments it takes."""
import numpy as np
import pytest
import torch

import paper_2209_05433_amd as fp8

pytestmark = pytest.mark.gpu

E4M3, E5M2 = fp8.FP8_E4M3, fp8.FP8_E5M2


def test_outputs_that_are_lazy_clones_leave_their_origin_alone():
    """A lazy clone shares memory with its origin until one of them is written: every tensor that a call writes gets
    memory of its own first."""
    x = torch.randn(64, 96, device="cuda")
    w = torch.randn(96, 32, device="cuda")
    f32 = lambda *s: torch.full(s, 7.0, device="cuda")
    u8 = lambda *s: torch.full(s, 7, dtype=torch.uint8, device="cuda")
    one, rows = torch.ones(1, device="cuda"), torch.ones(64, device="cuda")
    qx, qw = torch.zeros(64, 96, dtype=torch.uint8, device="cuda"), torch.zeros(96, 32, dtype=torch.uint8, device="cuda")
    ws = lambda n: torch.zeros(n * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")
    split = lambda: u8(max(4, fp8.fp8_gemm_splitk_workspace_size(64, 32, 96, False, False, 2)))
    calls = {
        "fp8_amax": ([f32(1)], lambda o: fp8.fp8_amax(x, o[0])),
        "fp8_amax_scale": ([f32(1), f32(1), ws(1)], lambda o: fp8.fp8_amax_scale(x, E4M3, *o)),
        "fp8_amax_scale_multi": ([f32(2), f32(2), ws(2)], lambda o: fp8.fp8_amax_scale_multi((x, w), (E4M3, E4M3), *o)),
        "fp8_quantize_multi": ([u8(64, 96), u8(96, 32)], lambda o: fp8.fp8_quantize_multi((x, w), (E4M3, E4M3), torch.ones(2, device="cuda"), o)),
        "fp8_scale_from_amax": ([f32(1)], lambda o: fp8.fp8_scale_from_amax(one, E4M3, o[0])),
        "fp8_scale_from_amax_n": ([f32(64)], lambda o: fp8.fp8_scale_from_amax_n(rows, E4M3, o[0])),
        "fp8_scale_from_amax_history": ([f32(1)], lambda o: fp8.fp8_scale_from_amax_history(rows, E4M3, o[0])),
        "fp8_quantize": ([u8(64, 96)], lambda o: fp8.fp8_quantize(x, E4M3, 1.0, o[0])),
        "fp8_quantize_dscale": ([u8(64, 96)], lambda o: fp8.fp8_quantize_dscale(x, E4M3, one, o[0])),
        "fp8_quantize_ex": ([u8(64, 96)], lambda o: fp8.fp8_quantize_ex(x, E4M3, 1.0, 0, o[0])),
        "fp8_quantize_amax": ([u8(64, 96), f32(1)], lambda o: fp8.fp8_quantize_amax(x, E4M3, one, *o)),
        "fp8_quantize_sr": ([u8(64, 96)], lambda o: fp8.fp8_quantize_sr(x, E4M3, 1.0, 5, o[0])),
        "fp8_dequantize": ([f32(64, 96)], lambda o: fp8.fp8_dequantize(qx, E4M3, 1.0, o[0])),
        "fp8_amax_rows": ([f32(64)], lambda o: fp8.fp8_amax_rows(x, o[0])),
        "fp8_quantize_rows": ([u8(64, 96)], lambda o: fp8.fp8_quantize_rows(x, E4M3, rows, o[0])),
        "fp8_quantize_transpose": ([u8(64, 96), u8(96, 64)], lambda o: fp8.fp8_quantize_transpose(x, E4M3, one, *o)),
        "fp8_gemm": ([f32(64, 32)], lambda o: fp8.fp8_gemm(qx, E4M3, 1.0, qw, E4M3, 1.0, o[0])),
        "fp8_gemm_dscale": ([f32(64, 32)], lambda o: fp8.fp8_gemm_dscale(qx, E4M3, one, qw, E4M3, one, o[0])),
        "fp8_gemm_mfma8": ([f32(64, 32)], lambda o: fp8.fp8_gemm_mfma8(qx, E4M3, 1.0, qw, E4M3, 1.0, o[0])),
        "fp8_gemm_mfma8_dscale": ([f32(64, 32)], lambda o: fp8.fp8_gemm_mfma8_dscale(qx, E4M3, one, qw, E4M3, one, o[0])),
        "fp8_gemm_ex": ([f32(64, 32)], lambda o: fp8.fp8_gemm_ex(qx, E4M3, False, qw, E4M3, False, o[0], 1.0, 1.0)),
        "fp8_gemm_splitk": ([f32(64, 32), split()], lambda o: fp8.fp8_gemm_splitk(qx, E4M3, False, qw, E4M3, False, o[0], 1.0, 1.0, o[1], 0, 2)),
        "fp8_gemm_splitk_static": ([f32(64, 32)], lambda o: fp8.fp8_gemm_splitk_static(qx, E4M3, False, qw, E4M3, False, o[0], 1.0, 1.0)),
        "fp8_gemm_fused": ([u8(64, 32), f32(1)], lambda o: fp8.fp8_gemm_fused(qx, E4M3, False, qw, E4M3, False, o[0], fp8.FP8_OUT_E4M3, one, one, None, o[1])),
        "fp8_scaled_gemm": ([u8(64, 96), u8(96, 32), f32(2), f32(2), ws(2), f32(64, 32)],
                            lambda o: fp8.fp8_scaled_gemm(x, E4M3, False, w, E4M3, False, *o)),
    }
    assert set(calls) == set(fp8.binding.TENSOR_CALLS)
    for name, (origins, call) in calls.items():
        before, clones, plain = [t.clone() for t in origins], [torch._lazy_clone(t) for t in origins], [t.clone() for t in origins]
        call(clones)
        call(plain)
        torch.cuda.synchronize()
        assert all(torch.equal(t, b) for t, b in zip(origins, before)), name
        assert all(torch.equal(c, p) for c, p in zip(clones, plain)), name


def test_arguments_that_stand_for_integers_and_numbers():
    """Whatever int() takes is taken for flags, slices, seeds, kinds, the formats of a list and stream handles, and
    whatever float() takes for factors."""
    x = torch.randn(300, 64, device="cuda")
    q, r = (torch.zeros(x.shape, dtype=torch.uint8, device="cuda") for _ in range(2))
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()

    def same():
        torch.cuda.synchronize()
        assert torch.equal(q, r) and bool(q.any())
        q.zero_(), r.zero_()
        torch.cuda.synchronize()

    fp8.fp8_quantize_sr(x, E4M3, 2.0, 77, q)
    fp8.fp8_quantize_sr(x, E4M3, np.float64(2.0), 77.0, r, np.int64(stream.cuda_stream))
    same()
    fp8.fp8_quantize_ex(x, E4M3, 2.0, fp8.FP8_QUANT_NOSAT, q, stream)
    fp8.fp8_quantize_ex(x, np.int32(E4M3), "2.0", float(fp8.FP8_QUANT_NOSAT), r, stream.cuda_stream)
    same()
    one = torch.ones(1, device="cuda")
    fp8.fp8_quantize_multi([x], [E5M2], one, [q])
    fp8.fp8_quantize_multi([x], [1.0], one, [r], float(0))
    same()
    a, b = q[:64].view(64, 64).fill_(0x38), r[:64].view(64, 64).fill_(0x38)
    c, d = torch.zeros(64, 64, device="cuda"), torch.zeros(64, 64, device="cuda")
    ws = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    fp8.fp8_gemm_splitk(a, E4M3, False, b, E4M3, False, c, 1.0, 1.0, ws, fp8.FP8_GEMM_MFMA8, 1)
    fp8.fp8_gemm_splitk(a, E4M3, 0, b, E4M3, "", d, 1, True, ws, np.float32(fp8.FP8_GEMM_MFMA8), "1")
    torch.cuda.synchronize()
    assert torch.equal(c, d) and bool((c == 64.0).all())
    with pytest.raises(TypeError):
        fp8.fp8_quantize(x, 0.0, 1.0, q)                     # a format is an integer

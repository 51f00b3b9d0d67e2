"""Sizes at which the vectorised kernels meet their edges: rows that end inside a vector, tiles that
reach over the matrix, tensors that start anywhere.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2209_05433_amd as fp8
from gpu_util import bf16_to_bits, knob, launches

pytestmark = pytest.mark.gpu

E4M3, E5M2 = fp8.FP8_E4M3, fp8.FP8_E5M2
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def source(n, dtype, off, seed=3):
    """n values that start `off` elements into a buffer, and the same on the host."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    buf = torch.randn(n + off, device="cuda", generator=g).mul_(30.0).to(DTYPES[dtype])
    x = buf[off:]
    return x, (bf16_to_bits(x) if dtype == "bf16" else x.cpu().numpy())


def inside(n, off):
    """An output of n bytes `off` bytes into a buffer of guard bytes."""
    buf = torch.full((n + off + 64,), 0xAA, dtype=torch.uint8, device="cuda")
    return buf, buf[off:off + n]


def guards_hold(buf, n, off):
    b = buf.cpu().numpy()
    return bool((b[:off] == 0xAA).all() and (b[off + n:] == 0xAA).all())


# the forms of the one-launch amax and cast: chunks of 64 KB to their last (256 in all), of 128 KB, of 160 KB, one more element than those hold
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 1024, 7168, 1024), ("bf16", 1023, 7169, 1027), ("bf16", 4096, 4095, 2048), ("bf16", 4096, 5825, 2048), ("bf16", 4097, 5824, 2049),
                                         ("f32", 1024, 3000, 2047), ("f32", 2048, 2048, 2048), ("f32", 2049, 2048, 2048)])
def test_one_launch_casts_of_larger_tensors(M, N, K, dtype):
    test_one_call_equals_the_separate_calls_at_every_size_of_its_casts(M, N, K, dtype)
    if M * K < 1 << 22:
        a, b = (torch.randn(s, device="cuda").to(DTYPES[dtype]) for s in ((M, K), (K, N)))
        outs = []
        for patience in (0, 1):
            ws = torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")
            qa, qb, c = (torch.zeros(s, dtype=t, device="cuda") for s, t in ((a.shape, torch.uint8), (b.shape, torch.uint8), ((M, N), torch.float32)))
            amax, scale = torch.zeros(2, device="cuda"), torch.zeros(2, device="cuda")
            with knob(fp8.FP8_KNOB_PATIENCE, patience):
                fp8.fp8_scaled_gemm(a, E4M3, False, b, E5M2, False, qa, qb, amax, scale, ws, c)
            torch.cuda.synchronize()
            assert not bool(ws.any())
            outs.append((qa, qb, c, amax, scale))
        assert all(torch.equal(x, y) for x, y in zip(*outs))
        assert outs[0][3].tolist() == [float(a.abs().max()), float(b.abs().max())]


# the forms of the one-launch amax and cast (workgroups, threads): chunks of 64 KB to their last (256 in all), of 128 KB, of 160 KB; one more
# element than those hold, in three launches
@pytest.mark.parametrize("dtype,M,N,K,form", [("bf16", 1024, 7168, 1024, (256, 512)), ("bf16", 1023, 7169, 1027, (130, 1024)), ("bf16", 4096, 4095, 2048, (256, 1024)),
                                              ("bf16", 4096, 5825, 2048, (249, 1024)), ("bf16", 4097, 5824, 2049, (249, 1024)), ("f32", 1024, 3000, 2047, (252, 1024)),
                                              ("f32", 2048, 2048, 2048, (256, 1024)), ("f32", 2049, 2048, 2048, None)])
def test_forms_of_the_one_launch_casts_with_and_without_waiting(M, N, K, dtype, form):
    a, b = (torch.randn(s, device="cuda").to(DTYPES[dtype]) for s in ((M, K), (K, N)))
    outs = []
    for patience in (0, 1):
        ws = torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")
        qa, qb, c = (torch.zeros(s, dtype=t, device="cuda") for s, t in ((a.shape, torch.uint8), (b.shape, torch.uint8), ((M, N), torch.float32)))
        amax, scale = torch.zeros(2, device="cuda"), torch.zeros(2, device="cuda")
        call = lambda: fp8.fp8_scaled_gemm(a, E4M3, False, b, E5M2, False, qa, qb, amax, scale, ws, c)
        with knob(fp8.FP8_KNOB_PATIENCE, patience):
            call()
            torch.cuda.synchronize()
            assert form is None or not bool(ws.any())
            ran = launches(call)
            assert ran[0] == form and len(ran) == 2 if form else len(ran) == 3, ran
        outs.append((qa, qb, c, amax, scale))
    assert all(torch.equal(x, y) for x, y in zip(*outs))
    assert outs[0][3].tolist() == [float(a.abs().max()), float(b.abs().max())]


# one tile; tiles and chunks with one vector more and less than a whole one; the smallest and the longest K; tiles that share their chunks unevenly
SCALED = [(8, 8, 8), (32, 32, 128), (40, 24, 136), (256, 256, 256), (24, 1000, 120), (1000, 40, 264), (72, 200, 1024), (8, 64, 512), (33, 65, 520), (9, 70, 127), (35, 97, 9), (257, 131, 131), (64, 33, 1021), (15, 1000, 250), (33, 65, 511)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", SCALED)
def test_scaled_product_in_one_launch_equals_the_separate_calls(M, N, K, transA, transB, dtype):
    """fp8_scaled_gemm of a few small tiles is one launch: every result bit for bit that of the separate calls, with and
    without waiting for the other workgroups, both modes, between guards, again and again on one workspace; an output that
    shares memory with an operand (which keeps the launches apart) too."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((K, M) if transA else (M, K), device="cuda", generator=g).mul_(7.0).to(DTYPES[dtype])
    b = torch.randn((N, K) if transB else (K, N), device="cuda", generator=g).to(DTYPES[dtype])
    a.view(-1)[-1], b.view(-1)[-1] = 900.0, -300.0
    if M > 8:
        a.view(-1)[3] = float("nan") if K == 120 else 0.0
    ws = torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")
    new = lambda n, dt: torch.full((n + 128,), 3, dtype=dt, device="cuda")
    cut = lambda t, *shape: t[64:t.numel() - 64].view(*shape)
    for out, flags in ((torch.float32, 0), (torch.bfloat16, fp8.FP8_GEMM_MFMA8)):
        def buffers():
            return [new(a.numel(), torch.uint8), new(b.numel(), torch.uint8), new(M * N, out), torch.zeros(2, device="cuda"), torch.zeros(2, device="cuda")]
        def views(t):
            return cut(t[0], *a.shape), cut(t[1], *b.shape), cut(t[2], M, N), t[3], t[4]
        qa, qb, c, amax, scale = views(buffers())
        fp8.fp8_amax_scale_multi((a, b), (E5M2, E4M3), amax, scale, torch.zeros_like(ws))
        fp8.fp8_quantize_multi((a, b), (E5M2, E4M3), scale, (qa, qb))
        fp8.fp8_gemm_ex(qa, E5M2, transA, qb, E4M3, transB, c, scale[0:1], scale[1:2], flags=flags)
        want = [t.clone() for t in (qa, qb, c, amax, scale)]
        for patience in (0, 1, 0):
            bufs = buffers()
            got = views(bufs)
            with knob(fp8.FP8_KNOB_PATIENCE, patience):
                fp8.fp8_scaled_gemm(a, E5M2, transA, b, E4M3, transB, got[0], got[1], got[3], got[4], ws, got[2], flags)
            torch.cuda.synchronize()
            assert not bool(ws.any())
            for x, y in zip(got, want):
                assert torch.equal(x.contiguous().view(torch.uint8), y.view(torch.uint8)), (out, patience)
            for t in bufs[:3]:
                assert bool((t[:64] == 3).all()) and bool((t[-64:] == 3).all())
    if M * N * 4 <= a.numel() * a.element_size():
        c_in_a = a.view(-1).view(torch.uint8)[:M * N * 4].view(torch.float32).view(M, N)
        qa, qb, c, amax, scale = views([new(a.numel(), torch.uint8), new(b.numel(), torch.uint8), new(M * N, torch.float32), torch.zeros(2, device="cuda"), torch.zeros(2, device="cuda")])
        fp8.fp8_scaled_gemm(a, E5M2, transA, b, E4M3, transB, qa, qb, amax, scale, ws, c)
        fp8.fp8_scaled_gemm(a, E5M2, transA, b, E4M3, transB, qa, qb, amax, scale, ws, c_in_a)
        assert torch.equal(c.contiguous().view(torch.uint8), c_in_a.contiguous().view(torch.uint8))


# bf16: rows at which a thread gets six vectors, and eight; fp32: rows too long for the one launch
MORE_SCALED = [(40, 96, 520), (72, 64, 768), (24, 56, 776)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", MORE_SCALED)
def test_scaled_product_in_one_launch_of_longer_rows(M, N, K, transA, transB, dtype):
    test_scaled_product_in_one_launch_equals_the_separate_calls(M, N, K, transA, transB, dtype)


# the last below and the first at 192 KB along K in all tiles; 200 tiles and 204; 230 and 240 where an operand is contiguous along a K that is no multiple of 16;
# 64 and 72 where K is short and neither is
LINE = [(568, 272, 600), (512, 480, 512), (512, 512, 192), (800, 256, 64), (544, 384, 64), (736, 320, 24), (960, 256, 24), (256, 256, 16), (288, 256, 16)]


def one_launch(M, N, K, transA, transB, dtype, small):
    """Whether fp8_scaled_gemm is one launch: small tiles of 32 x 32, whole rows of up to 2048 bytes, others of up to 1024, less
    than 192 KB along K in all tiles, and no more tiles than the launches apart take longer for."""
    esz = 2 if dtype == "bf16" else 4
    ragged = (M if transA else K) * esz % 16 or (K if transB else N) * esz % 16
    tiles = -(-M // 32) * -(-N // 32)
    along_k = not transA or transB
    most = 235 if along_k and K % 16 else 64 if not along_k and K <= 16 else 200
    return small and K * esz <= (1024 if ragged else 2048) and tiles <= most and tiles * K * esz < 192 << 10


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", SCALED + MORE_SCALED + LINE)
def test_which_scaled_products_are_one_launch(M, N, K, transA, transB, dtype):
    a, b = (torch.ones(s, device="cuda", dtype=DTYPES[dtype]) for s in ((K, M) if transA else (M, K), (N, K) if transB else (K, N)))
    qa, qb, c = (torch.zeros(s, dtype=t, device="cuda") for s, t in ((a.shape, torch.uint8), (b.shape, torch.uint8), ((M, N), torch.float32)))
    amax, scale = torch.zeros(2, device="cuda"), torch.zeros(2, device="cuda")
    ws = torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")
    small = fp8.fp8_gemm_form(qa, transA, qb, transB, c, fp8.FP8_OUT_F32) == fp8.FP8_FORM_SMALL_32x32
    assert small or (M, N, K) in LINE or K < 16          # (the tests of the one launch are tests of it)
    ran = launches(lambda: fp8.fp8_scaled_gemm(a, E4M3, transA, b, E4M3, transB, qa, qb, amax, scale, ws, c))
    assert len(ran) == (1 if one_launch(M, N, K, transA, transB, dtype, small) else 2), ran


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,cols,off", [(127, 255, 0), (129, 257, 1), (136, 264, 0), (8, 3, 1), (3, 8, 0), (257, 513, 3), (140, 126, 0), (128, 256, 1),
                                           # the line between tiles and one element per lane: few rows, few columns, few elements
                                           (11, 96001, 1), (12, 96001, 1), (81000, 13, 3), (81000, 14, 0), (1024, 256, 1), (1024, 257, 0), (1024, 1024, 0), (1025, 1025, 1),
                                           # tiles of 64, 128 and 256 columns, their last row of tiles a quarter, a half and nearly full
                                           (16384 + 30, 64, 0), (16384 + 33, 65, 1), (8192 + 64, 128, 0), (8192 + 100, 129, 1), (32, 40000, 0), (33, 40001, 3), (64, 20000, 1), (65, 20003, 0),
                                           (1100, 1003, 1), (1030, 1022, 0), (1027, 1029, 3)])
def test_transposing_cast_at_the_edges_of_its_tiles(rows, cols, off, dtype):
    n = rows * cols
    x, host = source(n, dtype, off)
    scale = torch.full((1,), 3.0, device="cuda")
    want = oracle.quantize(host.reshape(rows, cols), E4M3, np.float32(3.0))
    bq, q = inside(n, off)
    bt, qt = inside(n, off)
    fp8.fp8_quantize_transpose(x.view(rows, cols), E4M3, scale, q.view(rows, cols), qt.view(cols, rows))
    torch.cuda.synchronize()
    assert np.array_equal(q.view(rows, cols).cpu().numpy(), want)
    assert np.array_equal(qt.view(cols, rows).cpu().numpy(), want.T)
    assert guards_hold(bq, n, off) and guards_hold(bt, n, off)


# (M, N, K, offset of both operands in bytes): each form of the small-tile kernel, at one and several tiles, with
# rows shorter than a vector, K shorter than a chunk, K ends inside a chunk, and operands that start anywhere
SMALL = [(1, 1, 1, 0), (5, 15, 17, 0), (31, 33, 63, 1), (32, 32, 64, 0), (33, 63, 65, 3), (16, 320, 2048, 0), (17, 97, 1030, 5), (64, 130, 129, 0),
         (65, 1025, 127, 0), (100, 260, 1100, 7), (300, 1030, 200, 0), (257, 400, 2500, 1), (700, 900, 513, 0)]


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,off", SMALL)
def test_small_tiles_at_their_edges(M, N, K, off, transA, transB):
    """Small integers, so that every sum is exact in every order: all four outputs kinds and both
    instruction modes against the oracle, with guard words around the output."""
    rng = np.random.default_rng(M * 31 + N * 7 + K)
    A = oracle.quantize(rng.integers(-3, 4, (M, K)).astype(np.float32), E4M3, np.float32(1.0))
    B = oracle.quantize(rng.integers(-3, 4, (K, N)).astype(np.float32), E5M2, np.float32(1.0))
    S, _ = oracle.gemm_rows(A, E4M3, B, E5M2)

    def operand(x):
        buf, view = inside(x.size, off)
        view.copy_(torch.from_numpy(np.ascontiguousarray(x).reshape(-1)))
        return view.view(*x.shape)

    dA, dB = operand(A.T if transA else A), operand(B.T if transB else B)
    sA, sB, sD = torch.full((M,), 2.0, device="cuda"), torch.full((N,), 0.5, device="cuda"), torch.full((1,), 0.25, device="cuda")
    sA[M // 2] = 4.0
    c_ref = S / (sA.cpu().numpy().astype(np.float64)[:, None] * 0.5)
    amax = torch.full((1,), -1.0, device="cuda")
    for flags in (0, fp8.FP8_GEMM_MFMA8):
        for kind, dtype in ((fp8.FP8_OUT_F32, torch.float32), (fp8.FP8_OUT_BF16, torch.bfloat16), (fp8.FP8_OUT_E4M3, torch.uint8)):
            buf = torch.full((M * N + 16,), 9, dtype=dtype, device="cuda")
            D = buf[8:8 + M * N].view(M, N)
            fp8.fp8_gemm_fused(dA, E4M3, transA, dB, E5M2, transB, D, kind, sA, sB, sD if dtype == torch.uint8 else None, amax, flags)
            torch.cuda.synchronize()
            if dtype == torch.uint8:
                assert np.array_equal(D.cpu().numpy(), oracle.quantize(c_ref.astype(np.float32), E4M3, np.float32(0.25)))
            else:
                assert np.array_equal(D.double().cpu().numpy(), torch.from_numpy(c_ref).to(dtype).double().numpy())
            assert bool((buf[:8] == 9).all()) and bool((buf[8 + M * N:] == 9).all())
            assert float(amax.item()) == float(np.max(np.abs(c_ref)))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,off", [(1, 0), (7, 1), (15, 1), (16, 0), (4095, 3), (16 * 2048, 0), (16 * 2048 + 1, 1), (32 * 1024 + 5, 1), (262144 + 9, 0), (1048576 * 4 + 3, 1)])
def test_flat_casts_at_any_length_and_address(n, off, dtype):
    """amax and factor, plain cast, cast + amax, stochastic cast and back, on tensors that start
    anywhere and end inside a vector, an item or a chunk."""
    x, host = source(n, dtype, off, seed=n)
    ws = torch.zeros(fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")
    amax, scale, amax2 = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.full((1,), -1.0, device="cuda")
    for _ in range(2):
        fp8.fp8_amax_scale(x, E5M2, amax, scale, ws)
    a_ref = oracle.amax(host)
    s_ref = oracle.scale_from_amax(a_ref, E5M2)
    bufs = [inside(n, off) for _ in range(3)]
    fp8.fp8_quantize_dscale(x, E5M2, scale, bufs[0][1])
    fp8.fp8_quantize_amax(x, E5M2, scale, bufs[1][1], amax2)
    fp8.fp8_quantize_sr(x, E5M2, scale, 77, bufs[2][1])
    back = torch.full((n + 2,), 5.0, device="cuda")
    fp8.fp8_dequantize(bufs[0][1], E5M2, scale, back[1:1 + n])
    torch.cuda.synchronize()
    assert np.float32(amax.item()) == a_ref and np.float32(scale.item()) == s_ref and np.float32(amax2.item()) == a_ref
    want = oracle.quantize(host, E5M2, s_ref)
    assert np.array_equal(bufs[0][1].cpu().numpy(), want) and np.array_equal(bufs[1][1].cpu().numpy(), want)
    assert np.array_equal(bufs[2][1].cpu().numpy(), oracle.quantize_sr(host, E5M2, s_ref, 77))
    assert np.array_equal(back[1:1 + n].cpu().numpy(), oracle.dequantize(want, E5M2, s_ref).astype(np.float32))
    assert back[0].item() == 5.0 and back[n + 1].item() == 5.0
    assert all(guards_hold(b, n, off) for b, _ in bufs)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", [(1, 1, 3), (33, 65, 127), (256, 256, 256), (1, 100000, 7), (300, 5000, 300), (2049, 3000, 1025), (4096, 6144, 2048)])
def test_one_call_equals_the_separate_calls_at_every_size_of_its_casts(M, N, K, dtype):
    """fp8_scaled_gemm keeps operands of up to 40 MB (fp32: 32 MB) together in registers between amax and cast: one and several workgroups per tensor, ends inside a vector, twice on one workspace (the first call
    has to leave it as it found it), and a workspace the separate calls have used."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), device="cuda", generator=g).mul_(7.0).to(DTYPES[dtype])
    b = torch.randn((K, N), device="cuda", generator=g).to(DTYPES[dtype])
    a.view(-1)[-1] = 900.0                                # the largest values are the last ones
    b.view(-1)[-1] = -300.0
    new = lambda *shape, dt=torch.float32: torch.zeros(shape, dtype=dt, device="cuda")
    ws = new(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dt=torch.int32)
    amax, scale, qa, qb, c = new(2), new(2), new(M, K, dt=torch.uint8), new(K, N, dt=torch.uint8), new(M, N)
    fp8.fp8_amax_scale_multi((a, b), (E4M3, E5M2), amax, scale, ws)
    fp8.fp8_quantize_multi((a, b), (E4M3, E5M2), scale, (qa, qb))
    fp8.fp8_gemm_ex(qa, E4M3, False, qb, E5M2, False, c, scale[0:1], scale[1:2])
    for _ in range(3):
        amax1, scale1, qa1, qb1, c1 = new(2), new(2), new(M, K, dt=torch.uint8), new(K, N, dt=torch.uint8), new(M, N)
        fp8.fp8_scaled_gemm(a, E4M3, False, b, E5M2, False, qa1, qb1, amax1, scale1, ws, c1)
        torch.cuda.synchronize()
        assert torch.equal(amax, amax1) and torch.equal(scale, scale1)
        assert torch.equal(qa, qa1) and torch.equal(qb, qb1) and torch.equal(c, c1)
    assert amax1.tolist() == [900.0, 300.0]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", [(300, 1000, 300), (515, 129, 513), (1, 40000, 7)])
def test_one_launch_casts_without_waiting(M, N, K, dtype):
    """A workgroup of the one-launch amax and cast that stops waiting takes the missing maxima from the tensor: with no
    wait at all, several workgroups per tensor and ends inside a vector, on one workspace again and again;
    maxima, factors and bytes are the oracle's and the workspace is left cleared."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), device="cuda", generator=g).to(DTYPES[dtype])
    b = torch.randn((K, N), device="cuda", generator=g).to(DTYPES[dtype])
    a.view(-1)[-1], b.view(-1)[0] = 900.0, -300.0
    hosts = [bf16_to_bits(t).reshape(t.shape) if dtype == "bf16" else t.cpu().numpy() for t in (a, b)]
    ws = torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")
    amax, scale, c = torch.zeros(2, device="cuda"), torch.zeros(2, device="cuda"), torch.zeros((M, N), device="cuda")
    want = [(oracle.amax(h), oracle.scale_from_amax(oracle.amax(h), f)) for h, f in zip(hosts, (E4M3, E5M2))]
    with knob(fp8.FP8_KNOB_PATIENCE, 1):
        for _ in range(20):
            qa, qb = (torch.zeros(t.shape, dtype=torch.uint8, device="cuda") for t in (a, b))
            fp8.fp8_scaled_gemm(a, E4M3, False, b, E5M2, False, qa, qb, amax, scale, ws, c)
            torch.cuda.synchronize()
            assert not bool(ws.any())
            assert [(np.float32(x), np.float32(s)) for x, s in zip(amax.tolist(), scale.tolist())] == want
            for q, h, f, w in ((qa, hosts[0], E4M3, want[0]), (qb, hosts[1], E5M2, want[1])):
                assert np.array_equal(q.cpu().numpy(), oracle.quantize(h, f, w[1]))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,cols,off", [(1, 1, 1), (37, 3, 0), (5, 8, 1), (18, 121, 0), (70, 515, 1), (9, 2053, 0), (6, 3001, 3), (3, 4099, 0), (2, 20001, 1), (4, 8192, 0), (65, 256, 0), (5, 2048, 1), (7, 4096, 0), (3, 2052, 0)])
def test_rows_of_every_length(rows, cols, off, dtype):
    """Row maxima, factors and cast in each form (lanes per row), rows that start anywhere and end inside a
    vector; the largest value of a row is its last one."""
    n = rows * cols
    x, host = source(n, dtype, off, seed=rows)
    x = x.view(rows, cols)
    x[:, -1] = -500.0
    host = (bf16_to_bits(x) if dtype == "bf16" else x.cpu().numpy()).reshape(rows, cols)
    amax, scale = torch.full((rows,), -1.0, device="cuda"), torch.zeros(rows, device="cuda")
    buf, q = inside(n, off)
    fp8.fp8_amax_rows(x, amax)
    fp8.fp8_scale_from_amax_n(amax, E4M3, scale)
    fp8.fp8_quantize_rows(x, E4M3, scale, q.view(rows, cols))
    torch.cuda.synchronize()
    a_ref = oracle.amax_rows(host)
    assert np.array_equal(amax.cpu().numpy(), a_ref)
    assert np.array_equal(q.view(rows, cols).cpu().numpy(), oracle.quantize_rows(host, E4M3, oracle.scale_from_amax_n(a_ref, E4M3)))
    assert guards_hold(buf, n, off)

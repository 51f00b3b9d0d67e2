"""Two HIP streams and two host threads drive the library at once: the entry points keep no state
between calls (the amax cells are the callers', the error text is per thread), so every result must
equal the one obtained alone."""
import threading
import time

import numpy as np
import pytest
import torch

import paper_2209_05433_amd as fp8

pytestmark = pytest.mark.gpu

E4M3, E5M2 = fp8.FP8_E4M3, fp8.FP8_E5M2


def whole_path(x, w, fmt_x, out, stream, form, ws):
    """amax -> scale -> cast of both operands -> GEMM, all on `stream`; returns the intermediates.
    form "plain": one launch per step and tensor (atomic maximum in the caller's cell); "multi": amax +
    scale of both tensors in one launch and both casts in one launch, tickets in the workspace `ws`,
    which belongs to this stream alone."""
    amax = torch.zeros(2, device="cuda")
    scale = torch.zeros(2, device="cuda")
    qx = torch.empty(x.shape, dtype=torch.uint8, device="cuda")
    qw = torch.empty(w.shape, dtype=torch.uint8, device="cuda")
    if form == "multi":
        fp8.fp8_amax_scale_multi((x, w), (fmt_x, E4M3), amax, scale, ws, stream=stream)
        fp8.fp8_quantize_multi((x, w), (fmt_x, E4M3), scale, (qx, qw), stream=stream)
    else:
        for t, q, i, f in ((x, qx, 0, fmt_x), (w, qw, 1, E4M3)):
            fp8.fp8_amax(t, amax[i:i + 1], stream=stream)
            fp8.fp8_scale_from_amax(amax[i:i + 1], f, scale[i:i + 1], stream=stream)
            fp8.fp8_quantize_dscale(t, f, scale[i:i + 1], q, stream=stream)
    fp8.fp8_gemm_dscale(qx, fmt_x, scale[0:1], qw, E4M3, scale[1:2], out, stream=stream)
    return amax, scale, qx, qw


@pytest.mark.parametrize("form", ["plain", "multi"])
def test_two_streams_and_two_threads_give_the_single_stream_results(form):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    jobs = []
    for (M, N, K, fmt, dt) in ((1024, 1536, 2048, E4M3, torch.bfloat16), (768, 4096, 1024, E5M2, torch.float32)):
        x = torch.randn((M, K), device="cuda", generator=g).to(torch.bfloat16)
        w = (torch.randn((K, N), device="cuda", generator=g) * 0.02).to(torch.bfloat16)
        jobs.append((x, w, fmt, dt, (M, N)))
    torch.cuda.synchronize()
    # alone, on the default stream
    alone = []
    for x, w, fmt, dt, shape in jobs:
        out = torch.empty(shape, dtype=dt, device="cuda")
        mids = whole_path(x, w, fmt, out, None, form, torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        alone.append((out.clone(), [m.clone() for m in mids]))
    # together: one host thread and one stream per job, several rounds each
    streams = [torch.cuda.Stream() for _ in jobs]
    results = [None] * len(jobs)
    errors = []

    def worker(j):
        try:
            x, w, fmt, dt, shape = jobs[j]
            with torch.cuda.stream(streams[j]):
                ws = torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")    # this stream's own
                for _ in range(6):
                    out = torch.full(shape, 3.0, dtype=dt, device="cuda")
                    mids = whole_path(x, w, fmt, out, streams[j], form, ws)
                streams[j].synchronize()
                results[j] = (out, mids)
        except Exception as e:                                  # pragma: no cover
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(j,)) for j in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for j in range(len(jobs)):
        out, mids = results[j]
        ref_out, ref_mids = alone[j]
        assert torch.equal(out.view(torch.int16 if out.dtype == torch.bfloat16 else torch.int32),
                           ref_out.view(torch.int16 if out.dtype == torch.bfloat16 else torch.int32)), j
        for a, b in zip(mids, ref_mids):
            assert torch.equal(a, b), j


# one launch for all of the step; amax + cast in one launch: chunks of 64 KB, of 128 KB (bf16, fp32), of 160 KB.  From the third on
# four of them do not fit the chip together.
@pytest.mark.parametrize("M,N,K,dt", [(256, 256, 256, torch.float32), (1024, 1024, 1024, torch.bfloat16), (2048, 4096, 2048, torch.bfloat16),
                                      (2048, 2000, 2000, torch.float32), (2048, 6144, 2048, torch.bfloat16)])
def test_steps_whose_launches_wait_within_themselves_on_four_streams(M, N, K, dt):
    """fp8_scaled_gemm on four streams and threads at once, each with buffers and a workspace of its own: the results are
    those of a call alone, and no launch waits long for workgroups that another one keeps from running (a call takes
    no more than three times what the separate launches take in the same situation)."""
    g = torch.Generator(device="cuda").manual_seed(M + N)
    jobs, want = [], []
    for _ in range(4):
        a, b = (torch.randn(s, device="cuda", generator=g).to(dt) for s in ((M, K), (K, N)))
        outs = [torch.zeros(s, dtype=t, device="cuda") for s, t in (((M, K), torch.uint8), ((K, N), torch.uint8), ((M, N), torch.float32), ((2,), torch.float32), ((2,), torch.float32))]
        jobs.append((a, b, *outs, torch.zeros(2 * fp8.FP8_AMAX_WORKSPACE_BYTES // 4, dtype=torch.int32, device="cuda")))

    def one(a, b, qa, qb, c, amax, scale, ws):
        fp8.fp8_scaled_gemm(a, E4M3, False, b, E5M2, False, qa, qb, amax, scale, ws, c)

    def apart(a, b, qa, qb, c, amax, scale, ws):
        fp8.fp8_amax_scale_multi((a, b), (E4M3, E5M2), amax, scale, ws)
        fp8.fp8_quantize_multi((a, b), (E4M3, E5M2), scale, (qa, qb))
        fp8.fp8_gemm_ex(qa, E4M3, False, qb, E5M2, False, c, scale[0:1], scale[1:2])

    for j in jobs:
        apart(*j)
        torch.cuda.synchronize()
        want.append([t.clone() for t in j[2:7]])
        for t in j[2:]:                                     # (the separate launches leave partial maxima in the workspace)
            t.zero_()
    streams, errors, calls = [torch.cuda.Stream() for _ in jobs], [], 20

    def worker(i, f):
        try:
            with torch.cuda.stream(streams[i]):
                for _ in range(calls):
                    f(*jobs[i])
        except Exception as e:                                  # pragma: no cover
            errors.append(e)

    def together(f):
        """Seconds a call, the best of three times."""
        best = 1e9
        for _ in range(3):
            torch.cuda.synchronize()
            began = time.perf_counter()
            threads = [threading.Thread(target=worker, args=(i, f)) for i in range(len(jobs))]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - began) / calls)
        return best

    took = together(one)
    assert not errors, errors
    for j, w in zip(jobs, want):
        assert not bool(j[7].any())
        for x, y in zip(j[2:7], w):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))
    assert took < 3.0 * together(apart) + 50e-6, "%.0f us a call" % (1e6 * took)

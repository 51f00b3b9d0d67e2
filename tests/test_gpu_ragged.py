"""Sizes at which the vectorised kernels meet their edges: rows that end inside a vector, tiles that
reach over the matrix, tensors that start anywhere.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2209_05433_amd as fp8
from gpu_util import bf16_to_bits

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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,cols,off", [(127, 255, 0), (129, 257, 1), (136, 264, 0), (8, 3, 1), (3, 8, 0), (257, 513, 3), (140, 126, 0), (128, 256, 1)])
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

"""GPU: column sums (bias gradients) at the edges of their strips and row lanes, and whole-grid launches, which take wider
strips, against one-device launches bit for bit."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from bench import event_time_ms
from oracle import blocks
from workloads import round_to_bf16
from gpu_util import mat_to_dev, empty, dt, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("q,mb,nb", [(2, 1, 1), (2, 7, 9), (2, 129, 65), (4, 1025, 1024), (4, 300, 136), (1, 2048, 24), (2, 2049, 16), (4, 4100, 64),
                                       (4, 2600, 1032), (1, 9000, 8)])
def test_strips_rows_and_launch_shapes(q, mb, nb, dtype):
    M, N = mb * q, nb * q
    dY = np.random.default_rng(9).standard_normal((M, N)).astype(np.float32)
    dY = round_to_bf16(dY) if dtype == "bf16" else dY
    d = mat_to_dev(dY, q, dtype)
    grid, dev = empty(q * q * nb, "fp32"), empty(q * q * nb, "fp32")
    opt.bias_grad(d, grid, M, N, q, -1, -1, dt(dtype))
    for i in range(q):
        for j in range(q):
            opt.bias_grad(d, dev, M, N, q, i, j, dt(dtype))
    torch.cuda.synchronize()
    assert np.array_equal(to_host(grid), to_host(dev))
    got = to_host(grid).reshape(q, q, nb)
    for i in range(q):
        for j in range(q):
            blk = blocks.block(dY, q, i, j).astype(np.float64)
            # a chain of at most rows/128 + 3 + 16 fp32 additions per column
            bound = (mb / 128 + 20) * 2.0 ** -24 * np.abs(blk).sum(axis=0)
            assert np.all(np.abs(got[i, j] - blk.sum(axis=0)) <= bound)


def test_tall_narrow_blocks_keep_their_loads_in_flight():
    """16 blocks of [8192 x 64] against 16 of [1024 x 512], the same bytes: 10.8 and 4.5 us; with the row lanes of short blocks and
    strips of 8 columns 30 us."""
    q, ms = 4, {}
    X, out = torch.randn(16 * 8192 * 64, device="cuda:0").to(torch.bfloat16), torch.empty(q * q * 512, device="cuda:0")
    for mb, nb in ((8192, 64), (1024, 512)):
        ms[mb] = event_time_ms(lambda: opt.bias_grad(X, out, mb * q, nb * q, q, -1, -1, opt.BF16), 20, warm=2)
    assert ms[8192] <= 4 * ms[1024], ms

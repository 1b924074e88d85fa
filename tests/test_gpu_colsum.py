"""GPU: column sums (bias gradients) at the edges of their strips and row lanes, and whole-grid launches, which take wider
strips, against one-device launches bit for bit."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from oracle import blocks
from workloads import round_to_bf16
from gpu_util import mat_to_dev, empty, dt, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("q,mb,nb", [(2, 1, 1), (2, 7, 9), (2, 129, 65), (4, 1025, 1024), (4, 300, 136), (1, 2048, 24)])
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

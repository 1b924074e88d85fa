"""GPU: the product kernel for fp32 operands and for bf16 rows that start on no 16-byte boundary, at the sizes where its
tiles, its 16-byte loads and its slabs of 128 bytes of k are cut: against the oracle, and whole grid against one device
(which choose different tiles) bit for bit."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from oracle import summa
from oracle.metrics import rel_frobenius
from workloads import gemm_inputs
from gpu_util import mat_to_dev, mat_to_host, empty, dt, to_host

pytestmark = pytest.mark.gpu
# one rounding to bf16 (8 significant bits) is at most 2^-8 relative to the element; fp32 sums of at most 520 terms stay below 520 * 2^-24 = 3.1e-5
# of the sum of the terms' magnitudes in the worst case and near its square root in practice
TOL = {"bf16": 2.0 ** -8, "fp32": 1e-5}
SHAPES = [(1, 1, 1), (3, 2, 5), (7, 3, 130), (31, 33, 29), (32, 64, 32), (33, 65, 36), (64, 32, 64), (65, 127, 63), (100, 260, 97)]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
@pytest.mark.parametrize("mb,kp,nb", SHAPES)
def test_cut_tiles_chunks_and_slabs(form, mb, kp, nb, dtype):
    q = 2
    M, K, N = mb * q, kp * q, nb * q
    A, B = gemm_inputs(31, form, M, K, N, dtype, "n1", "n1")
    dA, dB = mat_to_dev(A, q, dtype), mat_to_dev(B, q, dtype)
    # NaN on both sides of the operands: an element from outside that entered a sum would show
    pad = torch.full((64,), float("nan"), dtype=dA.dtype, device="cuda:0")
    dA, dB = torch.cat([pad, dA, pad])[64:-64], torch.cat([pad, dB, pad])[64:-64]
    dC = empty(M * N, dtype)
    opt.summa(form, dA, dB, dC, M, K, N, q, -1, -1, dt(dtype))
    torch.cuda.synchronize()
    assert rel_frobenius(mat_to_host(dC, M, N, q), summa.product(form, A, B)) <= TOL[dtype]


@pytest.mark.parametrize("dtype,mb,kp,nb", [("fp32", 256, 72, 250), ("bf16", 256, 71, 251)])
@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
def test_tile_choice_changes_no_bit(form, dtype, mb, kp, nb):
    q = 4                                   # 16 blocks: 64-wide tiles; one block: 32-wide tiles
    M, K, N = mb * q, kp * q, nb * q
    A, B = gemm_inputs(32, form, M, K, N, dtype, "n1", "n1")
    dA, dB = mat_to_dev(A, q, dtype), mat_to_dev(B, q, dtype)
    grid, dev = empty(M * N, dtype), empty(M * N, dtype)
    opt.summa(form, dA, dB, grid, M, K, N, q, -1, -1, dt(dtype))
    for i in range(q):
        for j in range(q):
            opt.summa(form, dA, dB, dev, M, K, N, q, i, j, dt(dtype))
    torch.cuda.synchronize()
    assert np.array_equal(to_host(grid), to_host(dev))

"""GPU: the product kernel for fp32 operands and for bf16 rows that start on no 16-byte boundary, at the sizes where its
tiles, its 16-byte loads and its slabs of k are cut: against the oracle, and whole grid against one device
(which choose different tiles) bit for bit."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from bench import event_time_ms
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


# 16 blocks: slabs of 64 bytes of k (one, two, more per panel; a row shorter than a load); one block: slabs of 256
@pytest.mark.parametrize("dtype,mb,kp,nb", [("fp32", 260, 3, 257), ("fp32", 256, 16, 256), ("fp32", 261, 17, 258), ("fp32", 512, 32, 320),
                                            ("fp32", 520, 33, 500), ("fp32", 512, 96, 512), ("bf16", 259, 7, 263), ("bf16", 260, 36, 257),
                                            ("bf16", 515, 69, 517), ("bf16", 513, 131, 516)])
@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
def test_short_panels_in_launches_that_fill_the_chip(form, dtype, mb, kp, nb):
    q = 4
    M, K, N = mb * q, kp * q, nb * q
    A, B = gemm_inputs(33, form, M, K, N, dtype, "n1", "n1")
    # NaN on both sides of the operands, and an element's offset of them: no element from outside, no 16-byte alignment
    pad = torch.full((65,), float("nan"), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda:0")
    dA, dB = (torch.cat([pad, mat_to_dev(X, q, dtype), pad])[65:-65] for X in (A, B))
    grid, dev = empty(M * N, dtype), empty(M * N, dtype)
    opt.summa(form, dA, dB, grid, M, K, N, q, -1, -1, dt(dtype))
    for i in range(q):
        for j in range(q):
            opt.summa(form, dA, dB, dev, M, K, N, q, i, j, dt(dtype))
    torch.cuda.synchronize()
    assert np.array_equal(to_host(grid), to_host(dev))
    assert rel_frobenius(mat_to_host(grid, M, N, q), summa.product(form, A, B)) <= TOL[dtype]


def test_short_panels_cost_less_than_long_ones():
    """16 blocks of [1024 x 1024]: panels of 8 stay well below the time of panels of 64, to which slabs of 256 bytes pad them
    (0.3 of it measured; padded 1.08)."""
    q, mb = 4, 1024
    us = {}
    for kp in (8, 64):
        A = torch.randn(mb * kp * q * q, device="cuda:0")
        C = torch.empty(mb * mb * q * q, device="cuda:0")
        us[kp] = event_time_ms(lambda: opt.summa("ab", A, A, C, mb * q, kp * q, mb * q, q, -1, -1, opt.FP32), 10, warm=2)
    assert us[8] <= 0.6 * us[64], us

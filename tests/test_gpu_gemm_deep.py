"""The 64x64 tile with four stages of 64 k in LDS (launches of at most two workgroups per CU): contractions that fill the stages
partly, exactly and several times over, against the oracle and, bit for bit, against the same tile's four-slab ring."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from oracle import summa
from oracle.metrics import rel_frobenius
from workloads import gemm_inputs
from gpu_util import mat_to_dev, mat_to_host, empty

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
@pytest.mark.parametrize("q,K", [(1, 64), (1, 128), (1, 192), (1, 256), (1, 320), (2, 384), (2, 640), (1, 1088)])
def test_stages(form, q, K):
    M, N = 128 * q, 192 * q
    A, B = gemm_inputs(K, form, M, K, N, "bf16", "n1", "n1")
    dA, dB = mat_to_dev(A, q, "bf16"), mat_to_dev(B, q, "bf16")
    bias = torch.randn(N, device="cuda:0")
    out = []
    try:
        for variant in (7, 1007):
            opt.binding.debug_set_gemm_variant(variant)
            plain, act = empty(M * N, "bf16"), empty(M * N, "bf16")
            opt.summa(form, dA, dB, plain, M, K, N, q, -1, -1, opt.BF16)
            opt.summa_ex(form, dA, dB, act, M, K, N, q, -1, -1, opt.BF16, bias=bias, act=1)
            torch.cuda.synchronize()
            assert tuple(opt.binding.debug_last_gemm_plan())[0] == 7
            out.append((plain, act))
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    assert rel_frobenius(mat_to_host(out[0][0], M, N, q), summa.product(form, A, B)) <= 5e-3   # one rounding to bf16: 2^-9
    for x, y in zip(*out):
        assert torch.equal(x.view(torch.int16), y.view(torch.int16))

"""The 64x64 tile with four stages of 64 k in LDS (launches of at most two workgroups per CU): contractions that fill the stages
partly, exactly and several times over, against the oracle and, bit for bit, against the same tile's four-slab ring; the last
launch that takes it and the first that does not; partial tiles of a panel split, in either order of the workgroups."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from oracle import summa
from oracle.metrics import rel_frobenius
from workloads import gemm_inputs
from gpu_util import mat_to_dev, mat_to_host, empty

pytestmark = pytest.mark.gpu
TOL = 5e-3   # one rounding to bf16: 2^-9
RING = 1000  # + variant: the older k-loop


def _same_bits(x, y):
    return torch.equal(x.view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
@pytest.mark.parametrize("q,K", [(1, 64), (1, 128), (1, 192), (1, 256), (1, 320), (2, 384), (2, 640), (1, 1088)])
def test_stages(form, q, K):
    M, N = 128 * q, 192 * q
    A, B = gemm_inputs(K, form, M, K, N, "bf16", "n1", "n1")
    dA, dB = mat_to_dev(A, q, "bf16"), mat_to_dev(B, q, "bf16")
    bias = torch.randn(N, device="cuda:0")
    out = []
    try:
        for variant in (7, RING + 7):
            opt.binding.debug_set_gemm_variant(variant)
            plain, act = empty(M * N, "bf16"), empty(M * N, "bf16")
            for run in (lambda: opt.summa(form, dA, dB, plain, M, K, N, q, -1, -1, opt.BF16),
                        lambda: opt.summa_ex(form, dA, dB, act, M, K, N, q, -1, -1, opt.BF16, bias=bias, act=1)):
                run()
                tile, splits, walked = opt.binding.debug_last_gemm_plan()
                assert tile == 7
                assert opt.binding.debug_last_gemm_deep() == (variant == 7 and not walked), (splits, walked)
            torch.cuda.synchronize()
            out.append((plain, act))
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    assert rel_frobenius(mat_to_host(out[0][0], M, N, q), summa.product(form, A, B)) <= TOL
    for x, y in zip(*out):
        assert _same_bits(x, y)


@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
def test_two_workgroups_per_compute_unit_and_one_more(form):
    tiles = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    M, K = 64, 320
    for n, deep in ((tiles, True), (tiles + 1, False)):
        N = 64 * n
        A, B = gemm_inputs(n, form, M, K, N, "bf16", "n1", "n1")
        dA, dB = mat_to_dev(A, 1, "bf16"), mat_to_dev(B, 1, "bf16")
        out = []
        try:
            for variant in (7, RING + 7):
                opt.binding.debug_set_gemm_variant(variant)
                C = empty(M * N, "bf16")
                opt.summa(form, dA, dB, C, M, K, N, 1, -1, -1, opt.BF16)
                torch.cuda.synchronize()
                assert opt.binding.debug_last_gemm_plan() == (7, 1, 0)
                assert opt.binding.debug_last_gemm_deep() == (deep and variant == 7)
                out.append(C)
        finally:
            opt.binding.debug_set_gemm_variant(-1)
        assert _same_bits(*out)
        assert rel_frobenius(mat_to_host(out[0], M, N, 1), summa.product(form, A, B)) <= TOL


# one device's block [Mb x q*Kp x Nb]: panels of up to 16 MiB (tile after tile) and of more (range after range), four stages and the
# ring, 128x128 tiles, blocks that no tile divides
@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
@pytest.mark.parametrize("variant,Mb,Kp,Nb,q,deep", [(7, 128, 512, 192, 4, True), (7, 512, 1024, 512, 4, True), (7, 384, 3072, 384, 4, True),
                                                     (3, 256, 1024, 256, 4, False), (3, 512, 2048, 768, 4, False),
                                                     (7, 200, 328, 136, 4, False), (7, 392, 2808, 392, 4, False)])
def test_partial_tiles_of_a_split(form, variant, Mb, Kp, Nb, q, deep):
    M, K, N, i, j = q * Mb, q * Kp, q * Nb, 1, 2
    gen = torch.Generator(device="cuda:0").manual_seed(Mb + Kp)
    dA = torch.randn(M * K, device="cuda:0", generator=gen).to(torch.bfloat16)
    dB = torch.randn(K * N, device="cuda:0", generator=gen).to(torch.bfloat16)
    out = {}
    try:
        for loop in (0, RING):
            opt.binding.debug_set_gemm_variant(loop + variant)
            ws = torch.full((opt.summa_workspace_bytes(form, M, K, N, q, i, j, opt.BF16),), 0xFF, dtype=torch.uint8, device="cuda:0")
            for w in (ws, None):
                C = empty(M * N, "bf16")
                opt.summa(form, dA, dB, C, M, K, N, q, i, j, opt.BF16, ws=w)
                torch.cuda.synchronize()
                plan = opt.binding.debug_last_gemm_plan()
                assert plan[0] == variant and plan[1] > 1 and plan[2] == (w is None)
                assert opt.binding.debug_last_gemm_deep() == (deep and not loop and w is not None)
                out[loop, w is None] = C
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    got = out[0, False].view(q, q, Mb, Nb)
    for C in out.values():
        assert torch.equal(C.view(q, q, Mb, Nb)[i, j].view(torch.int16), got[i, j].view(torch.int16))
    assert torch.isnan(got[i, j]).sum() == 0 and torch.isnan(got).sum() == (q * q - 1) * Mb * Nb
    a = dA.view(q, q, Kp, Mb)[:, i].reshape(K, Mb).t() if form == "atb" else dA.view(q, q, Mb, Kp)[i].permute(1, 0, 2).reshape(Mb, K)
    b = dB.view(q, q, Nb, Kp)[j].permute(1, 0, 2).reshape(Nb, K).t() if form == "abt" else dB.view(q, q, Kp, Nb)[:, j].reshape(K, Nb)
    want = a.float().cpu().double() @ b.float().cpu().double()
    assert rel_frobenius(got[i, j].float().cpu().numpy(), want.numpy()) <= TOL


@pytest.mark.parametrize("tile,rows,cols", [(6, 128, 64), (3, 128, 128)])
@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
@pytest.mark.parametrize("q,K", [(1, 64), (1, 192), (1, 256), (1, 320), (2, 640)])
def test_wider_tiles(tile, rows, cols, form, q, K):
    """One workgroup of 128x64 or 128x128 per CU: stages filled partly, exactly and several times over; one tile too many takes the ring."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for n, deep in ((3, True), (cus // (q * q), True), (cus + 1, False)):
        M, N = rows * q, cols * n * q
        A, B = gemm_inputs(K + n, form, M, K, N, "bf16", "n1", "n1")
        dA, dB = mat_to_dev(A, q, "bf16"), mat_to_dev(B, q, "bf16")
        out = []
        try:
            for variant in (tile, RING + tile):
                opt.binding.debug_set_gemm_variant(variant)
                c = empty(M * N, "bf16")
                opt.summa(form, dA, dB, c, M, K, N, q, -1, -1, opt.BF16)
                got, splits, walked = opt.binding.debug_last_gemm_plan()
                assert got == tile
                assert opt.binding.debug_last_gemm_deep_wide() == (deep and variant == tile and not walked)
                torch.cuda.synchronize()
                out.append(c)
        finally:
            opt.binding.debug_set_gemm_variant(-1)
        assert _same_bits(*out)
        assert rel_frobenius(mat_to_host(out[0], M, N, q), summa.product(form, A, B)) <= TOL


# one device's block: the wider tiles in every range of a split, up to one workgroup on each of 256 CUs
@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
@pytest.mark.parametrize("variant,Mb,Kp,Nb,q", [(6, 256, 1024, 256, 4), (6, 1024, 1024, 512, 4), (3, 256, 1024, 256, 4), (3, 512, 2048, 768, 4)])
def test_wider_tiles_in_a_split(form, variant, Mb, Kp, Nb, q):
    M, K, N, i, j = q * Mb, q * Kp, q * Nb, 2, 1
    gen = torch.Generator(device="cuda:0").manual_seed(Mb + Nb)
    dA, dB = (torch.randn(n, device="cuda:0", generator=gen).to(torch.bfloat16) for n in (M * K, K * N))
    bias = torch.randn(N, device="cuda:0", generator=gen)
    out = []
    try:
        for loop in (0, RING):
            opt.binding.debug_set_gemm_variant(loop + variant)
            ws = torch.full((opt.summa_workspace_bytes(form, M, K, N, q, i, j, opt.BF16),), 0xFF, dtype=torch.uint8, device="cuda:0")
            C = empty(M * N, "bf16")
            opt.summa_ex(form, dA, dB, C, M, K, N, q, i, j, opt.BF16, bias=bias, act=1, ws=ws)
            tile, splits, walked = opt.binding.debug_last_gemm_plan()
            assert tile == variant and splits > 1 and not walked
            assert opt.binding.debug_last_gemm_deep_wide() == (not loop)
            torch.cuda.synchronize()
            out.append(C.view(q, q, Mb, Nb)[i, j])
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    assert _same_bits(out[0].contiguous(), out[1].contiguous()) and not torch.isnan(out[0]).any()


@pytest.mark.parametrize("form", ["ab", "abt", "atb"])
@pytest.mark.parametrize("variant", [3, 6])
def test_wider_tiles_with_every_epilogue(form, variant):
    M, K, N = 256, 320, 384
    gen = torch.Generator(device="cuda:0").manual_seed(variant)
    dA, dB, pre_in, res = (torch.randn(n, device="cuda:0", generator=gen).to(torch.bfloat16) for n in (M * K, K * N, M * N, M * N))
    bias = torch.randn(N, device="cuda:0", generator=gen)
    out = []
    try:
        for loop in (0, RING):
            opt.binding.debug_set_gemm_variant(loop + variant)
            pre, act, back, wide = empty(M * N, "bf16"), empty(M * N, "bf16"), empty(M * N, "bf16"), empty(M * N, "fp32")
            for C, epi in ((act, dict(bias=bias, pre_act=pre, act=1)), (back, dict(gelu_grad_of=pre_in, residual=res)), (wide, dict(out_fp32=True))):
                opt.summa_ex(form, dA, dB, C, M, K, N, 1, 0, 0, opt.BF16, **epi)
                assert opt.binding.debug_last_gemm_deep_wide() == (not loop)
            torch.cuda.synchronize()
            out.append((pre, act, back, wide))
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    for x, y in zip(*out):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)) and not torch.isnan(x.float()).any()


@pytest.mark.parametrize("variant,d", [(3, 128), (6, 128), (6, 64)])
def test_wider_tiles_along_the_diagonal(variant, d):
    """The causal products of the attention: tiles above the diagonal skipped, contractions that end or begin at it."""
    b, s, n = 1, 768 if d == 64 else 512, 2
    h = n * d
    gen = torch.Generator(device="cuda:0").manual_seed(d)
    qkv, d_attn = (torch.randn(m, device="cuda:0", generator=gen).to(torch.bfloat16) for m in (b * s * 3 * h, b * s * h))
    ws = torch.empty(opt.attention_workspace_bytes(b, s, h, n, 1), dtype=torch.uint8, device="cuda:0")
    out = []
    try:
        for loop in (0, RING):
            opt.binding.debug_set_gemm_variant(loop + variant)
            P, O, g = empty(b * n * s * s, "bf16"), empty(b * s * h, "bf16"), empty(b * s * 3 * h, "bf16")
            ws.fill_(0xFF)
            opt.attention_fwd(qkv, P, O, b, s, h, n, 1, 0, 0, True, opt.BF16, ws)
            assert opt.binding.debug_last_gemm_plan()[0] == variant and opt.binding.debug_last_gemm_deep_wide() == (not loop)
            ws.fill_(0xFF)
            opt.attention_bwd(qkv, P, d_attn, g, b, s, h, n, 1, 0, 0, True, opt.BF16, ws)
            assert opt.binding.debug_last_gemm_plan()[0] == variant and opt.binding.debug_last_gemm_deep_wide() == (not loop)
            torch.cuda.synchronize()
            out.append((P, O, g))
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    for x, y in zip(*out):
        assert _same_bits(x, y) and not torch.isnan(x.float()).any()

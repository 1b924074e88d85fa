"""GPU: the forms of the fused attention's kernels (64- and 128-row workgroups, both gradients in one grid or one after the
other) on both sides of the lines between them, sequence lengths that cut their tiles, against fp64 on the GPU; whole grid
against one device bit for bit."""
import math

import pytest
import torch

import paper_2104_05343_amd as opt
from bench import event_time_ms

pytestmark = pytest.mark.gpu
TOL = 5e-3   # bf16 operands and results, fp32 sums: the bound the other attention tests use


def _reference(qkv, dO, b, s, n, d, causal):
    Q, K, V = qkv.double().view(b, s, n, 3, d).permute(3, 0, 2, 1, 4)
    S = torch.matmul(Q, K.transpose(2, 3).contiguous()) / math.sqrt(d)
    if causal:
        S = S.masked_fill(torch.ones(s, s, dtype=torch.bool, device=S.device).triu(1), -math.inf)
    P = torch.softmax(S, dim=3)
    G = dO.double().view(b, s, n, d).permute(0, 2, 1, 3)
    O = torch.matmul(P, V)
    dP = torch.matmul(G, V.transpose(2, 3).contiguous())
    dS = P * (dP - (dP * P).sum(dim=3, keepdim=True))
    grads = (torch.matmul(dS, K) / math.sqrt(d), torch.matmul(dS.transpose(2, 3).contiguous(), Q) / math.sqrt(d),
             torch.matmul(P.transpose(2, 3).contiguous(), G))
    return O.permute(0, 2, 1, 3).reshape(b * s, n * d), torch.stack(grads).permute(1, 3, 2, 0, 4).reshape(b * s, n * 3 * d)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("b,n,s,d", [(1, 2, 1, 128), (2, 3, 65, 128), (16, 4, 129, 128), (32, 8, 130, 128), (64, 8, 63, 128),
                                     (32, 8, 193, 128), (33, 8, 250, 64), (8, 8, 1025, 64), (64, 8, 127, 64)])
def test_forms_against_fp64(b, n, s, d, causal):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(s + n)
    qkv = torch.randn(b * s, n * 3 * d, generator=g, device="cuda:0").to(torch.bfloat16)
    dO = torch.randn(b * s, n * d, generator=g, device="cuda:0").to(torch.bfloat16)
    O, dQKV = torch.full_like(dO, float("nan")), torch.full_like(qkv, float("nan"))
    lse = torch.full((b * n * s,), float("nan"), device="cuda:0")
    h = n * d
    ws = torch.empty(opt.attention_fused_workspace_bytes(b, s, h, n, 1), dtype=torch.uint8, device="cuda:0")
    opt.attention_fused_fwd(qkv, O, lse, b, s, h, n, 1, 0, 0, causal, opt.BF16)
    opt.attention_fused_bwd(qkv, O, lse, dO, dQKV, b, s, h, n, 1, 0, 0, causal, opt.BF16, ws)
    torch.cuda.synchronize()
    o64, g64 = _reference(qkv, dO, b, s, n, d, causal)
    assert ((O.double() - o64).norm() / o64.norm()).item() <= TOL
    if s == 1:   # one key: its probability is one and dQ, dK are zero up to the rounding of O
        dv = dQKV.double().view(b, n, 3, d)[:, :, 2]
        assert (dv - dO.double().view(b, n, d)).abs().max().item() == 0.0
    else:
        assert ((dQKV.double() - g64).norm() / g64.norm()).item() <= TOL


# b, n of the whole q = 2 grid.  Head width 128: one device on the wide side of the causal line, and without a mask in one
# grid where the whole grid runs one kind after the other; 64: either side of the launch's line
@pytest.mark.parametrize("b,n,s,d,causal", [(32, 16, 130, 128, True), (8, 8, 1025, 128, False), (16, 8, 300, 128, True), (16, 16, 250, 64, True),
                                            (32, 16, 100, 64, True), (8, 16, 520, 64, False)])
def test_whole_grid_equals_one_device(b, n, s, d, causal):
    q, h = 2, n * d
    g = torch.Generator(device="cuda:0")
    g.manual_seed(s)
    qkv = torch.randn(b * s * 3 * h, generator=g, device="cuda:0").to(torch.bfloat16)
    dO = torch.randn(b * s * h, generator=g, device="cuda:0").to(torch.bfloat16)
    ws = torch.empty(opt.attention_fused_workspace_bytes(b, s, h, n, q), dtype=torch.uint8, device="cuda:0")
    out = []
    for where in ([(-1, -1)], [(i, j) for i in range(q) for j in range(q)]):
        O, dQKV = torch.full_like(dO, float("nan")), torch.full_like(qkv, float("nan"))
        lse = torch.full((b * n * s,), float("nan"), device="cuda:0")
        for i, j in where:
            opt.attention_fused_fwd(qkv, O, lse, b, s, h, n, q, i, j, causal, opt.BF16)
            opt.attention_fused_bwd(qkv, O, lse, dO, dQKV, b, s, h, n, q, i, j, causal, opt.BF16, ws)
        torch.cuda.synchronize()
        out.append((O, lse, dQKV))
    assert not any(torch.isnan(t).any() for t in out[0])
    assert all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(*out))


@pytest.mark.parametrize("d,s", [(64, 16390), (128, 8200)])
def test_long_sequences_without_a_mask(d, s):
    """K and V of a matrix beyond an XCD's L2: its tiles run together.  Sampled rows of two heads against fp64."""
    n, h = 2, 2 * d
    g = torch.Generator(device="cuda:0")
    g.manual_seed(d)
    qkv = torch.randn(s, 3 * h, generator=g, device="cuda:0").to(torch.bfloat16)
    O, lse = torch.full((s, h), float("nan"), dtype=torch.bfloat16, device="cuda:0"), torch.full((n, s), float("nan"), device="cuda:0")
    opt.attention_fused_fwd(qkv, O, lse, 1, s, h, n, 1, 0, 0, 0, opt.BF16)
    torch.cuda.synchronize()
    assert not torch.isnan(O).any() and not torch.isnan(lse).any()
    rows = torch.cat([torch.arange(0, 4), torch.randint(0, s, (120,)), torch.arange(s - 4, s)]).to("cuda:0")
    for head in range(n):
        Q, K, V = (qkv[:, head * 3 * d + k * d:head * 3 * d + (k + 1) * d].double() for k in range(3))
        S = Q[rows] @ K.T.contiguous() / math.sqrt(d)
        want = torch.softmax(S, dim=1) @ V
        assert ((O[rows, head * d:(head + 1) * d].double() - want).norm() / want.norm()).item() <= TOL
        assert (lse[head, rows].double() - torch.logsumexp(S, dim=1)).abs().max().item() <= 1e-2


def test_one_tile_per_matrix_costs_no_more_with_a_mask():
    """512 matrices of s = 128, width 64: 38.4 us causal, 37.6 without a mask; both kinds in one grid 42.7."""
    b, n, s, d = 64, 8, 128, 64
    h = n * d
    qkv, dO = torch.randn(b * s, 3 * h, device="cuda:0").to(torch.bfloat16), torch.randn(b * s, h, device="cuda:0").to(torch.bfloat16)
    O, dQKV, lse = torch.empty_like(dO), torch.empty_like(qkv), torch.empty(b * n * s, device="cuda:0")
    ws = torch.empty(opt.attention_fused_workspace_bytes(b, s, h, n, 1), dtype=torch.uint8, device="cuda:0")
    ms = []
    for causal in (1, 0):
        opt.attention_fused_fwd(qkv, O, lse, b, s, h, n, 1, 0, 0, causal, opt.BF16)
        ms.append(min(event_time_ms(lambda: opt.attention_fused_bwd(qkv, O, lse, dO, dQKV, b, s, h, n, 1, 0, 0, causal, opt.BF16, ws), 20, warm=2)
                      for _ in range(3)))
    assert ms[0] <= 1.08 * ms[1], ms

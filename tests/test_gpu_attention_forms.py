"""GPU: the forms of the fused attention's kernels (64- and 128-row workgroups, both gradients in one grid or one after the
other) on both sides of the lines between them, sequence lengths that cut their tiles, against fp64 on the GPU."""
import math

import pytest
import torch

import paper_2104_05343_amd as opt

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
                                     (32, 8, 193, 128), (33, 8, 250, 64), (8, 8, 1025, 64)])
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

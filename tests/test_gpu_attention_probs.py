"""GPU parity of the attention that keeps the probabilities at the edges of its row and column tiles: head widths 64 and 128,
sequences of one 8-row piece up to several 128-row tiles, launches of few matrices (64-row workgroups) and of many (128-row)."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from oracle import attention as oatt
from oracle.metrics import rel_frobenius
from workloads import round_to_bf16
from gpu_util import mat_to_dev, mat_to_host, empty, to_host

pytestmark = pytest.mark.gpu
TOL = 5e-3   # two bf16 roundings (P or dS, then the result), 2^-9 each

# (sequences, s, heads, head width): 256 tiles of 128 rows and more make the 128-row workgroups, without a mask more than 256 of 64
SHAPES = [(2, 8, 2, 64), (1, 64, 1, 128), (1, 72, 2, 128), (2, 200, 1, 64), (32, 136, 4, 128), (16, 200, 8, 64), (22, 264, 4, 64), (2, 520, 3, 128),
          (2, 520, 8, 128), (6, 200, 12, 128), (6, 264, 8, 64), (4, 264, 8, 64)]
# long walks: 64-row and 128-row workgroups of either width
SHAPES += [(1, 2048, 6, 64), (1, 1032, 32, 64), (2, 1024, 8, 128), (1, 1024, 32, 128)]


def _workspace(b, s, n, d):
    # all bits set: a NaN in bf16 and in fp32
    return torch.full((opt.attention_workspace_bytes(b, s, n * d, n, 1),), 0xFF, dtype=torch.uint8, device="cuda:0")


def _attention(qkv, d_attn, b, s, n, d, causal):
    h, M = n * d, b * s
    ws = _workspace(b, s, n, d)
    P, O, G = empty(b * n * s * s, "bf16"), empty(M * h, "bf16"), empty(M * 3 * h, "bf16")
    x, dO = mat_to_dev(qkv, 1, "bf16"), mat_to_dev(d_attn, 1, "bf16")
    opt.attention_fwd(x, P, O, b, s, h, n, 1, 0, 0, causal, opt.BF16, ws)
    ws.fill_(0xFF)
    opt.attention_bwd(x, P, dO, G, b, s, h, n, 1, 0, 0, causal, opt.BF16, ws)
    torch.cuda.synchronize()
    return P, O, G


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("b,s,n,d", SHAPES)
def test_edges(b, s, n, d, causal):
    h, M = n * d, b * s
    rng = np.random.default_rng(s + d)
    qkv = round_to_bf16((rng.standard_normal((M, 3 * h)) * 2).astype(np.float32))
    d_attn = round_to_bf16(rng.standard_normal((M, h)).astype(np.float32))
    P, O, G = _attention(qkv, d_attn, b, s, n, d, causal)
    attn_o, probs_o = oatt.forward(qkv, b, s, n, causal)
    p = to_host(P).reshape(b, n, s, s)
    assert rel_frobenius(p, probs_o) <= TOL
    if causal:
        iu = np.triu_indices(s, 1)
        assert np.all(p[..., iu[0], iu[1]] == 0.0) and np.all(p[..., 0, 0] == 1.0)
    assert rel_frobenius(mat_to_host(O, M, h, 1), attn_o) <= TOL
    got, want = mat_to_host(G, M, 3 * h, 1), oatt.backward(qkv, d_attn, b, s, n, causal)
    part = (np.arange(3 * h) // d) % 3
    for k in range(3):   # P rounded to bf16 before the backward: a third rounding
        assert rel_frobenius(got[:, part == k], want[:, part == k]) <= 1.5 * TOL, k


@pytest.mark.parametrize("variant", [6, 3, 1])   # 128x64, 128x128, 256x128
@pytest.mark.parametrize("b,s,n,d", [(1, 512, 16, 128), (3, 768, 16, 128)])
def test_zeros_past_the_diagonal_for_every_tile_of_dk(variant, b, s, n, d):
    """dS is read past the diagonal by the product that makes dK, up to the end of its tile's rows: 64 to 256."""
    h, M = n * d, b * s
    rng = np.random.default_rng(variant)
    qkv = round_to_bf16(rng.standard_normal((M, 3 * h)).astype(np.float32))
    d_attn = round_to_bf16(rng.standard_normal((M, h)).astype(np.float32))
    P, _, want = _attention(qkv, d_attn, b, s, n, d, True)
    assert torch.isnan(want).sum() == 0
    x, dO, got = mat_to_dev(qkv, 1, "bf16"), mat_to_dev(d_attn, 1, "bf16"), empty(M * 3 * h, "bf16")
    opt.debug_set_gemm_variant(variant)
    try:
        opt.attention_bwd(x, P, dO, got, b, s, h, n, 1, 0, 0, True, opt.BF16, _workspace(b, s, n, d))
        torch.cuda.synchronize()
        assert opt.debug_last_gemm_plan()[0] == variant
    finally:
        opt.debug_set_gemm_variant(-1)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("b,s,n,d", [(2, 200, 4, 64), (32, 136, 4, 128)])
def test_probabilities_above_the_diagonal_are_not_read(b, s, n, d):
    """Gradients of Q and K do not depend on what P holds above the diagonal (that of V does: its product reads whole tiles)."""
    h, M = n * d, b * s
    rng = np.random.default_rng(s)
    qkv = round_to_bf16(rng.standard_normal((M, 3 * h)).astype(np.float32))
    d_attn = round_to_bf16(rng.standard_normal((M, h)).astype(np.float32))
    P, _, want = _attention(qkv, d_attn, b, s, n, d, True)
    upper = torch.triu(torch.ones(s, s, dtype=torch.bool, device="cuda:0"), 1)
    P.view(b * n, s, s).masked_fill_(upper, float("nan"))
    x, dO, got = mat_to_dev(qkv, 1, "bf16"), mat_to_dev(d_attn, 1, "bf16"), empty(M * 3 * h, "bf16")
    opt.attention_bwd(x, P, dO, got, b, s, h, n, 1, 0, 0, True, opt.BF16, _workspace(b, s, n, d))
    torch.cuda.synchronize()
    qk = torch.from_numpy(np.flatnonzero((np.arange(3 * h) // d) % 3 < 2)).to("cuda:0")
    assert torch.equal(got.view(torch.int16).view(M, -1)[:, qk], want.view(torch.int16).view(M, -1)[:, qk])


@pytest.mark.parametrize("s,d", [(136, 128), (200, 64)])
def test_workgroups_of_64_and_128_rows_same_bits(s, d):
    b, n = 16, 8   # 256 tiles of 128 rows; one sequence: 16
    h = n * d
    rng = np.random.default_rng(d)
    qkv = round_to_bf16(rng.standard_normal((b * s, 3 * h)).astype(np.float32))
    d_attn = round_to_bf16(rng.standard_normal((b * s, h)).astype(np.float32))
    P, O, G = _attention(qkv, d_attn, b, s, n, d, True)
    rows = slice(3 * s, 4 * s)
    P1, O1, G1 = _attention(qkv[rows], d_attn[rows], 1, s, n, d, True)
    assert torch.equal(P.view(torch.int16).view(b, -1)[3], P1.view(torch.int16))
    assert torch.equal(O.view(torch.int16).view(b, -1)[3], O1.view(torch.int16))
    cols = torch.from_numpy(np.flatnonzero((np.arange(3 * h) // d) % 3 == 0)).to("cuda:0")
    assert torch.equal(G.view(torch.int16).view(b * s, -1)[rows][:, cols], G1.view(torch.int16).view(s, -1)[:, cols])


def _peaked(b, s, n, d, rng):
    """qkv whose scores are the product of the first component of Q and of K, the rest small."""
    qkv = round_to_bf16((rng.standard_normal((b * s, 3 * n * d)) * 0.5).astype(np.float32))
    first = lambda part: (np.arange(n) * 3 + part) * d
    return qkv, first(0), first(1)


# Head width 64 and 128; 64-row and 128-row workgroups.
NONFINITE = [(1, 328, 2, 64), (32, 328, 4, 64), (1, 328, 8, 128), (32, 328, 4, 128)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("b,s,n,d", NONFINITE)
def test_blocks_of_minus_infinity(b, s, n, d, causal):
    """Scores that overflow to -inf weigh nothing, also where they are the first that a wavefront meets in a row."""
    rng = np.random.default_rng(5)
    qkv, q0, k0 = _peaked(b, s, n, d, rng)
    qkv[:, q0], qkv[:, k0] = 2.0 ** 66, 0.0
    rows = np.arange(b * s) % s
    qkv[np.ix_(rows < 128, k0)] = -2.0 ** 66   # the first block of either parity
    P, O, _ = _attention(qkv, np.ones((b * s, n * d), np.float32), b, s, n, d, causal)
    p = to_host(P).reshape(b, n, s, s)[:, :, 128:]
    assert np.all(p[..., :128] == 0.0)
    want = oatt.forward(qkv, b, s, n, causal)
    assert rel_frobenius(p, want[1][:, :, 128:]) <= TOL
    assert rel_frobenius(mat_to_host(O, b * s, n * d, 1)[rows >= 128], want[0][rows >= 128]) <= TOL


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("b,s,n,d", NONFINITE)
def test_scores_far_beyond_the_exponent(b, s, n, d, causal):
    """Finite scores of any size: a row's largest score weighs exp(0) however coarse the scores' last bit is."""
    rng = np.random.default_rng(6)
    qkv, q0, k0 = _peaked(b, s, n, d, rng)
    rows = np.arange(b * s) % s
    qkv[:, q0] = round_to_bf16((1e9 * (1 + rng.random((b * s, n)))).astype(np.float32))
    qkv[:, k0] = (rng.permutation(s)[rows] - s // 2)[:, None]   # distinct, exact in bf16: one key per row has all the weight
    P, O, G = _attention(qkv, np.ones((b * s, n * d), np.float32), b, s, n, d, causal)
    attn_o, probs_o = oatt.forward(qkv, b, s, n, causal)
    assert np.all((probs_o == 0.0) | (probs_o == 1.0))
    assert np.array_equal(to_host(P).reshape(b, n, s, s), probs_o)
    assert rel_frobenius(mat_to_host(O, b * s, n * d, 1), attn_o) <= TOL
    assert np.all(np.isfinite(mat_to_host(G, b * s, 3 * n * d, 1)))


@pytest.mark.parametrize("b,s,n,d", NONFINITE)
def test_infinite_last_value(b, s, n, d):
    """The rows past the end of V weigh nothing: an infinity in its last row comes through, and nothing else does."""
    rng = np.random.default_rng(7)
    qkv = round_to_bf16(rng.standard_normal((b * s, 3 * n * d)).astype(np.float32))
    clean = _attention(qkv, np.ones((b * s, n * d), np.float32), b, s, n, d, False)[1]
    last, col = np.arange(b * s) % s == s - 1, 2 * d + 5
    qkv[last, col] = np.inf
    got = mat_to_host(_attention(qkv, np.ones((b * s, n * d), np.float32), b, s, n, d, False)[1], b * s, n * d, 1)
    want = mat_to_host(clean, b * s, n * d, 1)
    want[:, 5] = np.inf
    assert np.array_equal(got, want)

"""The backward pass of a layer with both products of a linear layer in one launch: bit for bit what the separate launches give,
for split and unsplit products, cut tiles, both tile sizes, and a workspace full of NaN."""
import pytest
import torch

import paper_2104_05343_amd as opt
from workloads import LayerShape, layer_inputs
from layer_util import BWD_OUT, FP32_MATS, VEC_PART, alloc_layer

pytestmark = pytest.mark.gpu
SEPARATE = 1255   # automatic tiles with the older k-loop: the same bits, and no pairs


@pytest.mark.parametrize("shape,device,deep,tile", [
    (LayerShape(b=2, s=64, h=128, n=2, q=2), None, True, 7),       # whole grid, one or two tiles a block
    (LayerShape(b=2, s=64, h=256, n=4, q=2), (1, 0), True, 7),     # one device, two slabs a panel
    (LayerShape(b=1, s=512, h=512, n=8, q=1), (0, 0), True, 7),    # one panel: never split
    (LayerShape(b=4, s=512, h=512, n=8, q=4), (2, 1), True, 7),    # both products split
    (LayerShape(b=4, s=104, h=320, n=4, q=2), (0, 1), False, 7),   # cut tiles: 208 rows, 160 columns
    (LayerShape(b=2, s=1024, h=1024, n=8, q=1), (0, 0), None, None),    # long contractions, several workgroups per CU
    (LayerShape(b=4, s=1000, h=640, n=10, q=1), (0, 0), False, None),   # cut tiles, several workgroups per CU
    (LayerShape(b=2, s=1800, h=1024, n=8, q=1), (0, 0), False, 3),      # 128x128 tiles, cut
    (LayerShape(b=2, s=1792, h=1024, n=8, q=1), (0, 0), False, 3),      # 128x128 tiles
], ids=str)
def test_pairs_equal_separate_launches(shape, device, deep, tile):
    inp = layer_inputs(shape.s, shape, "bf16", perturb_affine=True)
    cfg, T, lt, ws = alloc_layer(inp, shape, True)
    assert opt.binding.debug_layer_bwd_streams(cfg, *(device or (-1, -1))) == 1
    opt.layer_fwd(cfg, lt, -1, -1, ws)
    names = BWD_OUT + FP32_MATS + list(VEC_PART)
    out = []
    try:
        for hook in (SEPARATE, -1):
            # the peers' blocks of every stage first; then the device's own pass
            opt.binding.debug_set_gemm_variant(SEPARATE)
            opt.layer_bwd(cfg, lt, -1, -1, ws)
            opt.binding.debug_set_gemm_variant(hook)
            ws.fill_(0xFF)   # NaN in fp32 and bf16
            opt.layer_bwd(cfg, lt, *(device or (-1, -1)), ws)
            assert opt.binding.debug_last_gemm_pair() == (hook == -1)
            if hook == -1:
                assert tile is None or opt.binding.debug_last_gemm_plan()[0] == tile
                assert deep is None or opt.binding.debug_last_gemm_deep() == deep
            torch.cuda.synchronize()
            out.append({n: T[n].clone() for n in names})
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    for n in names:
        assert not torch.isnan(out[1][n]).any(), n
        assert torch.equal(out[0][n], out[1][n]), n


@pytest.mark.parametrize("shape", [LayerShape(b=8, s=256, h=768, n=12, q=4), LayerShape(b=4, s=104, h=320, n=4, q=2)], ids=str)
@pytest.mark.parametrize("d_x", ["d_x", "d_out", "d_ln1_out"])
def test_workspace_without_room_and_gradient_in_place(shape, d_x):
    """The weight gradients' partial tiles do not fit: combined at once.  d_x in the place of a tensor that the column sums read."""
    inp = layer_inputs(3, shape, "bf16", perturb_affine=True)
    cfg, T, lt, ws = alloc_layer(inp, shape, True)
    opt.layer_fwd(cfg, lt, -1, -1, ws)
    opt.layer_bwd(cfg, lt, -1, -1, ws)
    i, j, q = 0, 1, shape.q

    def block(t):
        return t.view(q * q, -1)[i * q + j]
    names = [n for n in BWD_OUT + FP32_MATS + list(VEC_PART) if n not in (d_x, "d_x")]
    before = {n: T[n].clone() for n in ("d_out", "d_ln1_out")}
    opt.layer_bwd(cfg, lt, i, j, ws)
    torch.cuda.synchronize()
    want = {n: T[n].clone() for n in names}
    want_x = T["d_x"].clone()
    M, h = shape.M, shape.h
    products = [("abt", M, h, 4 * h), ("atb", 4 * h, M, h), ("abt", M, 4 * h, h), ("atb", h, M, 4 * h), ("abt", M, h, h), ("atb", h, M, h),
                ("abt", M, 3 * h, h), ("atb", h, M, 3 * h), ("ab", M, h, 3 * h), ("ab", M, h, h), ("ab", M, h, 4 * h), ("ab", M, 4 * h, h)]
    one = max(opt.summa_workspace_bytes(*p, q, c, c, opt.BF16) for p in products for c in (0, -1))
    least = opt.attention_workspace_bytes(shape.b, shape.s, h, shape.n, q) + 2 * ((one + 255) // 256 * 256)
    assert least < ws.numel() or shape.h != 768
    for n, t in before.items():
        T[n].copy_(t)
    for n in names:
        if n not in before:
            block(T[n]).fill_(float("nan"))
    lt2 = opt.make_layer_tensors({**T, "d_x": T[d_x]})
    opt.layer_bwd(cfg, lt2, i, j, ws[:least])
    torch.cuda.synchronize()
    assert torch.equal(block(T[d_x]), block(want_x))
    for n in names:
        assert torch.equal(block(T[n]), block(want[n])), n


# Products of y = x W in the order of the backward pass, [columns of x, columns of y] in units of h
LINEAR = [(4, 1), (1, 4), (1, 1), (1, 3)]


@pytest.mark.parametrize("shape,in_splits,w_splits", [
    (LayerShape(b=2, s=64, h=320, n=4, q=2), (1, 5, 1, 1), (1, 1, 1, 1)),      # a row's two wavefronts add five ranges each: a second trip
    (LayerShape(b=4, s=64, h=640, n=4, q=4), (1, 8, 1, 8), (1, 1, 1, 1)),      # four wavefronts, eight ranges, both LayerNorms
    (LayerShape(b=4, s=384, h=128, n=4, q=2), (1, 1, 1, 1), (6, 6, 6, 6)),     # four blocks of every weight gradient behind the column sums
    (LayerShape(b=4, s=384, h=144, n=6, q=2), (1, 1, 1, 1), (6, 6, 6, 6)),     # rows of 72 columns
], ids=str)
def test_partial_tiles_of_the_whole_grid(shape, in_splits, w_splits):
    """Splits that are not walked in a whole-grid pass: the LayerNorm that adds them for whole rows, their combines in the grid of the sums."""
    M, h, q = shape.M, shape.h, shape.q
    plan = opt.binding.debug_plan_summa
    for (k, n), x, w in zip(LINEAR, in_splits, w_splits):
        assert plan("abt", M, n * h, k * h, q, -1, -1)[1:] == (x, 0) and plan("atb", k * h, M, n * h, q, -1, -1)[1:] == (w, 0)
        assert opt.binding.debug_plan_pair(M, k * h, n * h, q, -1, -1)
    inp = layer_inputs(shape.s, shape, "bf16", perturb_affine=True)
    cfg, T, lt, ws = alloc_layer(inp, shape, True)
    assert opt.binding.debug_layer_bwd_streams(cfg, -1, -1) == 1
    opt.layer_fwd(cfg, lt, -1, -1, ws)
    names = BWD_OUT + FP32_MATS + list(VEC_PART) + ["bstats1", "bstats2"]
    out = []
    try:
        for hook in (SEPARATE, -1):
            opt.binding.debug_set_gemm_variant(hook)
            ws.fill_(0xFF)
            for n in names:
                T[n].fill_(float("nan"))
            opt.layer_bwd(cfg, lt, -1, -1, ws)
            assert opt.binding.debug_last_gemm_pair() == (hook == -1)
            torch.cuda.synchronize()
            out.append({n: T[n].clone() for n in names})
    finally:
        opt.binding.debug_set_gemm_variant(-1)
    ws.fill_(0xFF)
    opt.layer_bwd(cfg, lt, q - 1, 0, ws)     # one device's blocks again, the peers' as they are
    torch.cuda.synchronize()
    for n in names:
        assert not torch.isnan(out[1][n]).any(), n
        assert torch.equal(out[0][n], out[1][n]) and torch.equal(T[n], out[1][n]), n

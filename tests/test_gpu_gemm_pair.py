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

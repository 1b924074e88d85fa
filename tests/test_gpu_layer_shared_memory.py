"""The backward pass of a layer whose matrices share memory, each in the place of one that the pass no longer needs: bit for bit the
pass with memory for each, eager on one stream and where two would run, and captured."""
import pytest
import torch

import paper_2104_05343_amd as opt
from workloads import LayerShape, layer_inputs
from layer_util import BWD_OUT, FP32_MATS, VEC_PART, alloc_layer

pytestmark = pytest.mark.gpu

ORDER = ["d_pre_gelu", "d_w2", "d_ln2_out", "d_w1", "d_h_mid", "d_attn", "d_w_o", "d_qkv", "d_ln1_out", "d_w_qkv", "d_x"]
# what is written later: where it lies
PLACES = [{"d_attn": "d_ln2_out"}, {"d_attn": "xhat2"}, {"d_ln1_out": "d_ln2_out"}, {"d_ln1_out": "d_attn"}, {"d_attn": "gelu"},
          {"d_h_mid": "d_out"}, {"d_h_mid": "d_ln2_out"}, {"d_qkv": "d_pre_gelu"}, {"d_pre_gelu": "pre_gelu"}, {"d_w2": "pre_gelu"},
          {"d_w1": "gelu"}, {"d_x": "ln1_out"}, {"d_x": "d_pre_gelu"}, {"d_x": "d_ln1_out"}, {"d_x": "d_out"}, {"d_x": "d_h_mid"},
          {"d_h_mid": "d_out", "d_attn": "d_ln2_out", "d_qkv": "d_pre_gelu", "d_ln1_out": "d_ln2_out", "d_x": "d_out"}]
# streams of the pass with memory for each; blocks of more than 1 Mi elements have their column sums on the way where two streams run
SHAPES = [(LayerShape(b=2, s=256, h=128, n=2, q=1), 1, (0, 0), True), (LayerShape(b=4, s=128, h=256, n=4, q=2), 1, (-1, -1), False),
          (LayerShape(b=4, s=1024, h=512, n=8, q=1), 1, (0, 0), True), (LayerShape(b=1, s=2048, h=256, n=4, q=1), 2, (0, 0), True),
          (LayerShape(b=1, s=8256, h=192, n=3, q=1), 2, (-1, -1), True)]


def _span(t):
    return t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()


@pytest.fixture(scope="module", params=SHAPES, ids=lambda p: f"{p[0].b}x{p[0].s}x{p[0].h}-q{p[0].q}-streams{p[1]}")
def layer(request):
    shape, streams, device, fused = request.param
    cfg, T, lt, ws = alloc_layer(layer_inputs(shape.s, shape, "bf16", perturb_affine=True), shape, True, fused=fused)
    assert opt.binding.debug_layer_bwd_streams(cfg, *device) == streams
    opt.layer_fwd(cfg, lt, -1, -1, ws)
    given = {n: T[n].clone() for n in ("d_out", "gelu", "pre_gelu", "xhat2", "ln1_out")}
    opt.layer_bwd(cfg, lt, *device, ws)
    torch.cuda.synchronize()
    return cfg, T, ws, device, given, {n: T[n].clone() for n in BWD_OUT + FP32_MATS + list(VEC_PART)}


@pytest.mark.parametrize("captured", [False, True], ids=["eager", "captured"])
@pytest.mark.parametrize("place", PLACES, ids=lambda p: ",".join(f"{n}:{w}" for n, w in p.items()))
def test_bits_do_not_depend_on_shared_memory(layer, place, captured):
    cfg, T, ws, device, given, want = layer
    for start in (True, False):   # of the place
        U = dict(T)
        for n, w in place.items():
            mem, size = T[w].view(torch.uint8), T[n].numel() * T[n].element_size()
            assert size <= mem.numel()
            U[n] = (mem[:size] if start else mem[-size:]).view(T[n].dtype)
        for n in want:
            T[n].fill_(float("nan"))
        for n, t in given.items():
            T[n].copy_(t)
        lt = opt.make_layer_tensors(U)
        if captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                opt.layer_bwd(cfg, lt, *device, ws)
            graph.replay()
        else:
            opt.layer_bwd(cfg, lt, *device, ws)
        torch.cuda.synchronize()
        lost = {n for k, n in enumerate(ORDER) for m in ORDER[k + 1:] if _span(U[n])[0] < _span(U[m])[1] and _span(U[m])[0] < _span(U[n])[1]}
        for n in want:
            assert n in lost or torch.equal(U[n].view(torch.uint8), want[n].view(torch.uint8)), (start, n)


def test_sharing_that_needs_no_care_keeps_the_pairs():
    """d_x anywhere, d_ln1_out in the place of d_attn, d_pre_gelu in place: one stream, both products of a linear layer in one launch."""
    shape = LayerShape(b=2, s=256, h=128, n=2, q=1)
    cfg, T, lt, ws = alloc_layer(layer_inputs(1, shape, "bf16"), shape, True)
    opt.layer_fwd(cfg, lt, -1, -1, ws)
    for place, pairs in (({}, True), ({"d_x": "d_out"}, True), ({"d_ln1_out": "d_attn", "d_pre_gelu": "pre_gelu"}, True), ({"d_attn": "d_ln2_out"}, False)):
        opt.layer_bwd(cfg, opt.make_layer_tensors({**T, **{n: T[w] for n, w in place.items()}}), 0, 0, ws)
        assert opt.binding.debug_last_gemm_pair() == pairs, place
    torch.cuda.synchronize()

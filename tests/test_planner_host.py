"""Host logic of the product planner (no GPU: the plan is arithmetic on shapes; without a device the planner assumes
256 compute units).  The panel split is the only part of a plan that changes the bits of a result (it fixes the order
in which the panels' contributions are added), so it must be a function of ONE device's block shape alone: the same
for device mode and grid mode, with and without a co-running product, with and without workspace.  The tile may differ."""
import ctypes
import shutil
import subprocess
import threading

import pytest
import torch

import paper_2104_05343_amd as opt
from bench import layer_gemm_list
from workloads import CONFIGS, gemm_cases

plan = opt.binding.debug_plan_summa


def _products():
    out = []
    for name in ("config2", "config4", "config5"):
        shp = CONFIGS[name]["layer"]
        for (g, form, M, K, N) in layer_gemm_list(shp.b, shp.s, shp.h):
            out.append((f"{name}.{g}", form, M, K, N, shp.q))
    for c in gemm_cases("config3"):
        out.append((f"config3.{c.name}", c.form, c.M, c.K, c.N, c.q))
    return out


PRODUCTS = _products()


@pytest.mark.parametrize("case", PRODUCTS, ids=[p[0] for p in PRODUCTS])
def test_panel_split_depends_on_the_block_shape_only(case):
    _, form, M, K, N, q = case
    base = plan(form, M, K, N, q, 0, 0)
    assert base[1] >= 1
    for (i, j) in ((q - 1, 1 % q), (-1, -1)):
        for corun in (0, 1, 2):
            for have_ws in (True, False):
                p = plan(form, M, K, N, q, i, j, corun, have_ws)
                assert p[1] == base[1], (i, j, corun, have_ws, p, base)
                if not have_ws and p[1] > 1:
                    assert p[2] == 1          # no workspace: the split is walked inside the workgroups
                    assert p[0] not in (0, 4)  # the 256x256 tile has no registers for a second accumulator set


# panels up to the 2 GiB that the loads of a full tile reach from its corner (k-strided operand: panel length times row
# length; k-contiguous: rows of the tile times row length): the same plan as a little shorter
@pytest.mark.parametrize("form,M,K,N,shorter", [("atb", 4096, 23168, 23168, 23104), ("ab", 4096, 23168, 2048, 23104),
                                                ("atb", 1024, 65536, 16384, 65472), ("ab", 4096, 131072, 4096, 131008)])
def test_panels_inside_the_load_window_take_a_full_tile(form, M, K, N, shorter):
    p = plan(form, M, K, N, 1, 0, 0)
    assert p[0] != 5 and p == plan(form, M, shorter, N, 1, 0, 0)


# longer panels: the tiles that walk a panel in several windows, not the any-shape kernel
@pytest.mark.parametrize("form,M,K,N,q", [("atb", 1024, 65600, 16384, 1), ("ab", 2048, 65536, 32768, 1), ("atb", 128, 80000, 66048, 2),
                                          ("atb", 8192, 8192, 151936, 1), ("atb", 4194368, 128, 256, 1), ("ab", 512, 1024, 4194368, 1)])
def test_panels_beyond_the_load_window(form, M, K, N, q):
    assert plan(form, M, K, N, q, 0, 0)[0] in (3, 6, 7)


# few tiles and long panels, or rows far apart: the any-shape kernel
@pytest.mark.parametrize("form,M,K,N", [("ab", 512, 32768, 1024), ("abt", 1024, 1 << 20, 1024), ("atb", 64, 65600, 16384), ("abt", 1024, 4194368, 1024)])
def test_few_tiles_of_panels_over_a_gib(form, M, K, N):
    assert plan(form, M, K, N, 1, 0, 0)[0] == 5


# Long contractions in several panels, outputs of about one 128x64 tile per CU: split, where one workgroup would walk 256 slabs; up to 6144 not.
@pytest.mark.parametrize("split,form,Mb,K,Nb,q", [(True, "atb", 384, 8192, 4096, 2), (True, "atb", 768, 8192, 2048, 4), (True, "atb", 512, 8192, 4096, 8),
                                                  (True, "abt", 3072, 8192, 512, 4), (True, "abt", 384, 8192, 4096, 2), (True, "ab", 512, 8192, 4096, 8),
                                                  (False, "abt", 2048, 6144, 1024, 4), (False, "ab", 768, 4096, 2048, 8), (False, "atb", 512, 4096, 3072, 2)])
def test_split_of_long_contractions(split, form, Mb, K, Nb, q):
    variant, splits, _ = plan(form, Mb * q, K, Nb * q, q, 0, 0)
    assert (splits > 1) == split
    assert split or variant == 6


# one panel: 144 workgroups of 128x64 with a long contraction give way to 288 of 64x64, 160 and shorter ones do not
@pytest.mark.parametrize("variant,form,M,K,N", [(7, "ab", 768, 12288, 1536), (7, "abt", 3072, 16384, 384), (6, "ab", 768, 6144, 1536), (6, "ab", 640, 8192, 2048)])
def test_tile_of_long_contractions_in_one_panel(variant, form, M, K, N):
    assert plan(form, M, K, N, 1, 0, 0) == (variant, 1, 0)


def test_no_split_without_panels_and_errors():
    # q = 1: one panel, nothing to split
    assert plan("ab", 2048, 4096, 1024, 1, 0, 0)[1] == 1
    # a skinny long-K product of the 64-device grid shape splits, a square one does not
    sk = [c for c in gemm_cases("config3") if c.name == "mlp_down.ab"][0]      # block [2048 x 1536 x 384] x 8 panels
    assert plan(sk.form, sk.M, sk.K, sk.N, sk.q, 0, 0)[1] > 1
    shp = CONFIGS["config4"]["layer"]
    assert plan("ab", shp.M, shp.h, 4 * shp.h, shp.q, 1, 2)[1] == 1
    with pytest.raises(opt.OptimusError):
        plan("ab", 2048, 4096, 1000, 3, 0, 0)            # not divisible by q
    with pytest.raises(opt.OptimusError):
        plan("ab", 2048, 4096, 1024, 4, 4, 0)            # coordinate outside the grid
    with pytest.raises(opt.OptimusError):
        plan("ab", 36, 36, 36, 4, 0, 0)                  # blocks of 9: not a matrix-core shape


# q, b, s, h, n, fused: short passes, then passes whose products are small and whose attention is long, or both are large
@pytest.mark.parametrize("streams,shape", [(1, (4, 8, 512, 1024, 16, 0)), (1, (4, 8, 512, 1024, 16, 1)), (1, (2, 4, 64, 128, 4, 0)),
                                           (1, (2, 2, 2048, 512, 8, 1)), (1, (1, 1, 1024, 512, 8, 1)),
                                           (2, (4, 4, 4096, 256, 4, 1)), (2, (4, 4, 4096, 512, 8, 0)), (2, (4, 4, 16384, 256, 4, 1)),
                                           (2, (2, 2, 4096, 256, 4, 0)), (2, (4, 8, 2048, 512, 8, 0)), (2, (1, 1, 2048, 256, 4, 1)),
                                           (2, (4, 8, 1024, 4096, 32, 1))])
def test_streams_of_an_eager_backward_pass(streams, shape):
    q, b, s, h, n, fused = shape
    cfg = opt.LayerCfg(b, s, h, n, q, 1e-5, 1, opt.BF16, fused)
    assert opt.binding.debug_layer_bwd_streams(cfg, 0, 0) == streams


def test_streams_of_the_whole_grid_and_refused_arguments():
    cfg = opt.LayerCfg(8, 512, 1024, 16, 4, 1e-5, 1, opt.BF16, 0)
    assert opt.binding.debug_layer_bwd_streams(cfg, -1, -1) == 2      # 16 devices' products
    assert opt.binding.debug_layer_bwd_streams(cfg, 4, 0) == -1
    assert opt.binding.debug_layer_bwd_streams(opt.LayerCfg(8, 512, 1024, 15, 4, 1e-5, 1, opt.BF16, 0), 0, 0) == -1


# Lines of the stream rule: cut blocks at any size, one device as a grid, wide blocks that 128 does not divide, linear layers whose products do not go
# together.  Last column: the whole grid.
@pytest.mark.parametrize("streams,shape,grid", [
    (1, (1, 8, 1001, 4096, 32, 1), False), (1, (4, 4, 4100, 4096, 32, 1), False), (2, (4, 4, 16400, 256, 4, 1), False), (1, (4, 4, 16400, 1024, 16, 1), False),
    (1, (1, 1, 1536, 128, 2, 1), False), (1, (1, 8, 1001, 1024, 16, 1), False), (1, (1, 8, 1001, 1024, 16, 1), True), (1, (1, 1, 4100, 512, 8, 1), False), (1, (1, 1, 4100, 512, 8, 1), True),
    (1, (1, 16, 1024, 1600, 25, 1), False), (1, (4, 32, 1024, 3840, 60, 1), False), (2, (4, 32, 1024, 2304, 36, 1), False), (2, (4, 16, 1024, 4096, 32, 1), False),
    (2, (4, 16, 512, 1536, 24, 1), False), (2, (4, 16, 512, 1792, 28, 1), False), (1, (4, 8, 512, 1536, 24, 1), False), (1, (4, 32, 512, 1024, 16, 1), False),
    (2, (4, 8, 333, 512, 8, 1), True), (1, (4, 4, 512, 512, 8, 1), True), (2, (4, 8, 512, 512, 8, 1), True)])
def test_lines_of_the_stream_rule(streams, shape, grid):
    q, b, s, h, n, fused = shape
    cfg = opt.LayerCfg(b, s, h, n, q, 1e-5, 1, opt.BF16, fused)
    assert opt.binding.debug_layer_bwd_streams(cfg, *((-1, -1) if grid else (0, 0))) == streams


SWITCH_HOOK = """
extern void optimus_debug_set_gemm_variant(int);
void switch_hook(volatile int* stop) { while (!*stop) { optimus_debug_set_gemm_variant(3); optimus_debug_set_gemm_variant(-1); } }
"""


@pytest.fixture
def switched_hook(tmp_path):
    """A callable that runs another one while a second thread forces the 128x128 tile and lets it go, over and over."""
    if not shutil.which("gcc"):
        pytest.skip("needs a C compiler")
    src, so = tmp_path / "switch_hook.c", tmp_path / "switch_hook.so"
    src.write_text(SWITCH_HOOK)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), str(src), opt.binding.LIB_PATH], check=True)
    opt.lib()
    helper = ctypes.CDLL(str(so))

    def run(f):
        stop = ctypes.c_int(0)
        switching = threading.Thread(target=helper.switch_hook, args=(ctypes.byref(stop),))
        switching.start()
        try:
            return f()
        finally:
            stop.value = 1
            switching.join()
            opt.debug_set_gemm_variant(-1)
    return run


# The plans a thread keeps are those of the hooks they are filed under, also where another thread changes a hook meanwhile.
def test_kept_plans_belong_to_their_hooks(switched_hook):
    shapes = [("ab", 4 * 64 * m, 4 * 512, 4 * 64 * n, 4, 0, 0) for m in range(3, 13) for n in range(3, 13)]
    plans = {}

    def ask(key):
        plans[key] = [plan(*s) for s in shapes]

    def ask_while_and_after():
        switched_hook(lambda: ask("while"))
        ask("after")

    for target, args in ((ask, ("alone",)), (ask_while_and_after, ())):   # a thread each: plans are kept per thread
        t = threading.Thread(target=target, args=args)
        t.start()
        t.join()
    assert plans["after"] == plans["alone"]


# A launch never writes partial tiles beyond the workspace it was given, whatever the hooks say by then.  (Without a device the
# launch itself is refused; the plan it was refused with stays readable.)
@pytest.mark.skipif(torch.cuda.is_available(), reason="the operands are no memory")
def test_partial_tiles_fit_the_workspace_under_changing_hooks(switched_hook):
    M, K, N, q = 4 * 512, 4 * 1024, 4 * 512, 4
    need = {}
    for variant in (-1, 3):
        opt.debug_set_gemm_variant(variant)
        need[variant] = opt.summa_workspace_bytes("ab", M, K, N, q, 0, 0, opt.BF16)
    opt.debug_set_gemm_variant(-1)
    small = min(need.values())
    assert 0 < small < max(need.values())
    one, seen = ctypes.c_void_p(256), set()

    def launches():
        for _ in range(20000):
            opt.lib().optimus_summa_ab(one, one, one, M, K, N, q, 0, 0, opt.BF16, one, small, None)
            seen.add(opt.binding.debug_last_gemm_plan())
    switched_hook(launches)
    assert len(seen) >= 2
    for _, splits, walked in seen:
        assert walked or splits == 1 or 4 * splits * (M // q) * (N // q) <= small, seen


# M, K, N, q of y = x W: small blocks, one of which may be cut, and blocks with tiles of 128x128 share a launch; large ones whose 64x64 tiles
# would, or whose own tiles are twice as wide, and one long workgroup per CU beside many short ones do not
@pytest.mark.parametrize("pair,shape", [(True, (4096, 4096, 1024, 4)), (True, (1024, 512, 2048, 2)), (True, (8000, 1280, 5120, 4)), (True, (8008, 2048, 8192, 2)),
                                        (True, (8192, 16384, 4096, 4)), (False, (8192, 15360, 3840, 4)), (False, (32000, 8192, 2048, 4)),
                                        (False, (8192, 5376, 1344, 1)), (False, (4096, 8192, 2048, 1)), (False, (8192, 1536, 6144, 4)),
                                        (False, (2048, 2048, 6144, 2)), (True, (4096, 768, 3072, 2)), (False, (4096, 2048, 8192, 1))])
def test_pairs_of_a_layer_backward(pair, shape):
    M, K, N, q = shape
    assert opt.binding.debug_plan_pair(M, K, N, q, q - 1, 0) == pair
    with pytest.raises(opt.OptimusError):
        opt.binding.debug_plan_pair(0, K, N, q, 0, 0)

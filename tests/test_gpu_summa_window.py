"""GPU: bf16 products whose panels lie around and beyond the 2 GiB that one buffer resource of the loads covers: full tiles
with offsets up to its end, the ragged form that walks a panel in several windows (one and several panels, panel split in
memory and inside the workgroups), rows far apart.  Operands of -1, 0 and 1: every sum is exact in fp32."""
import pytest
import torch

import paper_2104_05343_amd as opt

pytestmark = pytest.mark.gpu


def _ternary(rows, cols, seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    out = torch.empty(rows, cols, dtype=torch.bfloat16, device="cuda:0")
    step = max(1, (1 << 27) // cols)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        out[r:r + n] = torch.randint(-1, 2, (n, cols), generator=g, device="cuda:0", dtype=torch.int8)
    return out


def _want(form, A, B, k):
    """sum over k in pieces, fp32 (exact), of blocks as they are stored"""
    C = 0
    step = max(1, (1 << 27) // max(A.numel() // k, B.numel() // k))
    for a in range(0, k, step):
        b = min(k, a + step)
        x = A[a:b].T if form == "atb" else A[:, a:b]
        y = B[:, a:b].T if form == "abt" else B[a:b]
        C = C + x.float().contiguous() @ y.float().contiguous()
    return C


# form, q, block rows, panel length, block columns, whether the tile divides the block and a panel fits one window
CASES = [("atb", 1, 256, 65536, 16384, True),     # B fills the window but for 32 KiB
         ("abt", 1, 256, 131072, 8320, True),     # 2 GiB of k-contiguous rows
         ("atb", 1, 72, 65600, 16456, False),     # two windows, edges cut
         ("ab", 1, 72, 65600, 16456, False),
         ("atb", 2, 64, 40000, 33024, False),     # two panels of two windows each, panel split
         ("atb", 1, 4194312, 40, 72, False),      # k rows of A 8 MB apart
         ("ab", 1, 40, 72, 4194312, False)]


@pytest.mark.parametrize("form,q,mb,kp,nb,whole", CASES)
def test_panels_around_the_window(form, q, mb, kp, nb, whole):
    i, j = q - 1, 0
    shapes = {"ab": ((mb, kp), (kp, nb)), "abt": ((mb, kp), (nb, kp)), "atb": ((kp, mb), (kp, nb))}[form]
    A, B = (_ternary(q * q * r, c, k) for k, (r, c) in enumerate(shapes))    # block-major: block (r, c) after block
    M, K, N = q * mb, q * kp, q * nb
    ws = torch.empty(max(256, opt.summa_workspace_bytes(form, M, K, N, q, i, j, opt.BF16)), dtype=torch.uint8, device="cuda:0")
    C = torch.full((q * q, mb, nb), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    opt.summa(form, A, B, C, M, K, N, q, i, j, opt.BF16, ws=ws)
    plan = opt.binding.debug_last_gemm_plan()
    assert plan[0] != 5 and (whole or plan[0] in (3, 6, 7)), plan
    (ra, _), (rb, _) = shapes
    want = 0
    for l in range(q):
        a = {"ab": i * q + l, "abt": i * q + l, "atb": l * q + i}[form]
        b = {"ab": l * q + j, "abt": j * q + l, "atb": l * q + j}[form]
        want = want + _want(form, A[a * ra:(a + 1) * ra], B[b * rb:(b + 1) * rb], kp)
    want = want.to(torch.bfloat16)
    assert torch.equal(C[i * q + j], want)
    if plan[1] > 1:     # the same split walked inside the workgroups
        C.fill_(float("nan"))
        opt.summa(form, A, B, C, M, K, N, q, i, j, opt.BF16)
        assert opt.binding.debug_last_gemm_plan()[2] == 1
        assert torch.equal(C[i * q + j], want)

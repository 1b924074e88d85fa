"""GPU: the embedding gradient where its sort and its runs are cut: one row for all tokens, runs that end and begin at the
wavefronts' parts, more than one chunk of tokens, widths that are no multiple of four, against sums in 64 bits."""
import numpy as np
import pytest
import torch

import paper_2104_05343_amd as opt
from workloads import round_to_bf16
from gpu_util import mat_to_dev, empty, dt, to_host

pytestmark = pytest.mark.gpu


def _tokens(kind, M, v, rng):
    if kind == "one":
        return np.full(M, v // 2, dtype=np.int32)
    if kind == "two":                       # neighbours in the same workgroup's rows, alternating
        return (v // 2 + (np.arange(M) & 1)).astype(np.int32)
    if kind == "outside":                   # clamped to the table
        return rng.integers(-3, v + 3, M).astype(np.int32)
    return np.minimum(rng.zipf(1.2, M) - 1, v - 1).astype(np.int32)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("kind", ["one", "two", "zipf", "outside"])
@pytest.mark.parametrize("q,rows,vb,hb", [(1, 1, 1, 1), (2, 33, 31, 6), (2, 2100, 70, 260), (1, 4097, 33, 5)])
def test_against_64_bit_sums(q, rows, vb, hb, kind, dtype):
    rng = np.random.default_rng(rows + hb)
    M, v, h = q * rows, q * vb, q * hb
    tok = _tokens(kind, M, v, rng)
    dX = rng.standard_normal((M, h)).astype(np.float32)
    dX = round_to_bf16(dX) if dtype == "bf16" else dX
    d, t = mat_to_dev(dX, q, dtype), torch.from_numpy(tok).to("cuda:0")
    grid, dev = empty(v * h, "fp32"), empty(v * h, "fp32")
    opt.embedding_bwd(t, d, grid, M, v, h, q, -1, -1, dt(dtype))
    for l in range(q):
        for j in range(q):
            opt.embedding_bwd(t, d, dev, M, v, h, q, l, j, dt(dtype))
    torch.cuda.synchronize()
    assert np.array_equal(to_host(grid), to_host(dev))
    want, mag = np.zeros((v, h)), np.zeros((v, h))
    np.add.at(want, np.clip(tok, 0, v - 1), dX.astype(np.float64))
    np.add.at(mag, np.clip(tok, 0, v - 1), np.abs(dX).astype(np.float64))
    got = to_host(grid).reshape(q, q, vb, hb).transpose(0, 2, 1, 3).reshape(v, h)
    # longest chain of fp32 additions to an element: a part's tokens (a 64th of a chunk's, at least four), then two for each part that meets in
    # the row, chunk after chunk: below M + 96 at these sizes
    assert np.all(np.abs(got - want) <= (M + 96) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("vb,hb", [(128, 64), (129, 65), (127, 132), (300, 4)])
@pytest.mark.parametrize("M", [63, 256, 257, 2 * 4096 + 3])
def test_edges_of_a_workgroups_rows_columns_and_parts(vb, hb, M):
    """128 rows, 64 columns; parts of exactly four entries and of more; a third chunk of three tokens; rows nobody names are zeros."""
    rng = np.random.default_rng(vb + M)
    tok = rng.integers(0, vb, M).astype(np.int32)
    tok[tok == 5] = 6
    tok[rng.random(M) < 0.3] = vb - 1
    dX = round_to_bf16(rng.standard_normal((M, hb)).astype(np.float32))
    out = torch.full((vb * hb + 1,), float("nan"), device="cuda:0")
    for shift in (0, 1):   # 16-byte aligned rows, and not
        o = out[shift:shift + vb * hb]
        opt.embedding_bwd(torch.from_numpy(tok).to("cuda:0"), mat_to_dev(dX, 1, "bf16"), o, M, vb, hb, 1, 0, 0, opt.BF16)
        torch.cuda.synchronize()
        want, mag = np.zeros((vb, hb)), np.zeros((vb, hb))
        np.add.at(want, tok, dX.astype(np.float64))
        np.add.at(mag, tok, np.abs(dX).astype(np.float64))
        got = to_host(o).reshape(vb, hb)
        # at most one fp32 addition per token and two per part and chunk that meet in a row
        assert np.all(np.abs(got - want) <= (M + 3 * 128) * 2.0 ** -24 * mag)
        assert not got[5].any()

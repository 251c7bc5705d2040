"""Calibration statistics where a query or a key holds a NaN or an infinity: rows of the map that do not exist as numbers
are counted nowhere (NaN < eps is false), the other rows as ever, and keys past the last token change no count."""
import numpy as np
import pytest

from oracle import paro_calibration as pc
from oracle import paro_oracle as po

pytestmark = pytest.mark.gpu

EPS, TIE = 1e-3, 2e-4


@pytest.mark.parametrize("block,d,grid", [(64, 64, (3, 5, 7)), (64, 128, (5, 9, 8)), (32, 64, (3, 5, 7)), (32, 128, (2, 9, 15))])
@pytest.mark.parametrize("where", ["q", "k"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_counts_and_sums(block, d, grid, where, value):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(1, 1, d, *grid, 0, block)
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    assert n % block
    gen = torch.Generator().manual_seed(n + d)
    q, k = (torch.randn((1, 1, n, d), generator=gen).to(torch.bfloat16) for _ in range(2))
    (q if where == "q" else k)[0, 0, 70, 3] = value
    with np.errstate(invalid="ignore"):
        p = pc.attention_map(q[0, 0].float().numpy(), k[0, 0].float().numpy())
    z = dict(device="cuda:0")
    q, k = q.to("cuda:0"), k.to("cuda:0")
    q16, k16 = (torch.empty(pb.codes_shape(s, 16, pb.PARO_ROWS), dtype=torch.bfloat16, **z) for _ in range(2))
    sc = torch.empty((1, 1, kb), dtype=torch.float32, **z)
    rows = torch.zeros((pb.paro_calib_row_stats_bytes(s),), dtype=torch.uint8, **z)
    for ids in ([0], [3]):
        ids = np.array(ids, np.uint8)
        pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, q, q16, sc)
        pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, k, k16, sc)
        if not ids.any():
            pb.paro_calib_row_stats(s, q16, k16, rows)
        with np.errstate(invalid="ignore"):
            ref = pc.block_stats(pc.reorder_map(p, po.perm_index(*grid, 0, int(ids[0]))), block, EPS, TIE)
        for form in ("one call", "from rows"):
            out = [torch.full((1, 1, kb, kb), -1, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
            if form == "one call":
                pb.paro_calib_block_stats(s, q16, k16, EPS, *out)
            else:
                pb.paro_calib_block_stats_from_rows(s, ids, q16, k16, rows, EPS, *out)
            bsum, _, bcnt = (x[0, 0].cpu().numpy() for x in out)
            assert np.all(bcnt >= ref["cnt_lo"]) and np.all(bcnt <= ref["cnt_hi"]), (form, ids)
            assert np.allclose(bsum, ref["sum"], rtol=TIE, atol=1e-30, equal_nan=True), (form, ids)


@pytest.mark.parametrize("block,d", [(64, 64), (64, 128), (32, 64), (32, 128)])
@pytest.mark.parametrize("dead", [slice(0, 64), slice(0, 130), slice(100, 192)])
def test_keys_of_minus_infinity(block, d, dead):
    """Every logit of the first block, of more than two blocks and of the last keys is minus infinity: those entries are 0."""
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(1, 1, d, 3, 8, 8, 0, block)
    n, kb = 192, 192 // block
    gen = torch.Generator().manual_seed(d)
    q, k = (torch.randn((1, 1, n, d), generator=gen).to(torch.bfloat16) for _ in range(2))
    q[..., 3] = 1.0
    k[:, :, dead, 3] = -float("inf")
    p = pc.attention_map(q[0, 0].float().numpy(), k[0, 0].float().numpy())
    ref = pc.block_stats(p, block, EPS, TIE)
    z = dict(device="cuda:0")
    q, k = q.to("cuda:0"), k.to("cuda:0")  # whole blocks: the operands in the default order are the tensors themselves
    rows = torch.zeros((pb.paro_calib_row_stats_bytes(s),), dtype=torch.uint8, **z)
    pb.paro_calib_row_stats(s, q, k, rows)
    for form in ("one call", "from rows"):
        out = [torch.full((1, 1, kb, kb), -1, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
        if form == "one call":
            pb.paro_calib_block_stats(s, q, k, EPS, *out)
        else:
            pb.paro_calib_block_stats_from_rows(s, np.zeros(1, np.uint8), q, k, rows, EPS, *out)
        bsum, bmax, bcnt = (x[0, 0].cpu().numpy() for x in out)
        assert np.allclose(bsum, ref["sum"], rtol=TIE, atol=1e-30) and np.allclose(bmax, ref["max"], rtol=TIE, atol=1e-30), form
        assert np.all(bcnt >= ref["cnt_lo"]) and np.all(bcnt <= ref["cnt_hi"]), form

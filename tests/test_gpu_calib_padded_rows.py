"""Calibration where the sequence does not fill its last block and the last token's logits are far below zero (a common
offset of K against an opposed query): the rows past the last token do not exist, whatever the statistics of the row
before them."""
import numpy as np
import pytest

from oracle import paro_calibration as pc
from oracle import paro_oracle as po

pytestmark = pytest.mark.gpu

EPS, SIGMA, ALPHA, DENSITY = 1e-3, 0.9, 0.5, 0.4
REL = 2e-4  # fp32 sums over N terms and logits of some 300 octaves, each good to a few 2^-24 of its size


def _inputs(n, d, logit, seed):
    """q, k [1, 2, n, d] as bf16 values: random, K around a common offset, the last query of both heads opposed to it."""
    import torch

    gen = torch.Generator().manual_seed(seed)
    q, k = (torch.randn((1, 2, n, d), generator=gen) for _ in range(2))
    q[..., n - 1, :] = -1.0
    k += logit / d ** 0.5
    return tuple(x.to(torch.bfloat16) for x in (q, k))


GRIDS = [(64, 64, (3, 5, 7), 0), (64, 128, (5, 9, 8), 0), (32, 64, (3, 5, 7), 0), (32, 128, (2, 9, 15), 0), (64, 64, (2, 8, 8), 41), (64, 64, (13, 20, 19), 0)]


@pytest.mark.parametrize("block,d,grid,text", GRIDS)
@pytest.mark.parametrize("logit", [100.0, 200.0])
def test_block_statistics(block, d, grid, text, logit):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(1, 2, d, *grid, text, block)
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    assert n % block
    q, k = _inputs(n, d, logit, n + d)
    maps = [pc.attention_map(q[0, h].float().numpy(), k[0, h].float().numpy()) for h in range(2)]
    last = (q[0, :, n - 1].double()[:, None] @ k[0].double().transpose(1, 2)) / d ** 0.5
    assert float(last.max()) < -80.0
    z = dict(device="cuda:0")
    q, k = q.to("cuda:0"), k.to("cuda:0")
    q16, k16 = (torch.empty(pb.codes_shape(s, 16, pb.PARO_ROWS), dtype=torch.bfloat16, **z) for _ in range(2))
    sc = torch.empty((1, 2, kb), dtype=torch.float32, **z)
    rows = torch.zeros((pb.paro_calib_row_stats_bytes(s),), dtype=torch.uint8, **z)
    for ids in ([0, 0], [4, 1]):
        ids = np.array(ids, np.uint8)
        pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, q, q16, sc)
        pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, k, k16, sc)
        if not ids.any():
            pb.paro_calib_row_stats(s, q16, k16, rows)
        for form in ("one call", "from rows"):
            out = [torch.full((1, 2, kb, kb), -1, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
            if form == "one call":
                pb.paro_calib_block_stats(s, q16, k16, EPS, *out)
            else:
                pb.paro_calib_block_stats_from_rows(s, ids, q16, k16, rows, EPS, *out)
            bsum, bmax, bcnt = (x[0].cpu().numpy() for x in out)
            for h in range(2):
                ref = pc.block_stats(pc.reorder_map(maps[h], po.perm_index(*grid, text, int(ids[h]))), block, EPS, REL)
                assert np.allclose(bsum[h], ref["sum"], rtol=REL, atol=1e-30), (form, ids, h)
                assert np.allclose(bmax[h], ref["max"], rtol=REL, atol=1e-30), (form, ids, h)
                assert np.all(bcnt[h] >= ref["cnt_lo"]) and np.all(bcnt[h] <= ref["cnt_hi"]), (form, ids, h)


@pytest.mark.parametrize("block,d,grid,text", GRIDS)
def test_whole_calibration(block, d, grid, text):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import calibrate

    s = pb.make_shape(1, 2, d, *grid, text, block)
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    k_img = -(-(n - text) // block)
    q, k = _inputs(n, d, 150.0, n + d + 1)
    r = calibrate(s, q.to("cuda:0"), k.to("cuda:0"), EPS, SIGMA, ALPHA, DENSITY)
    bsum = r["block_sum"][0].cpu().numpy()
    mq = r["m_quant"].cpu().numpy()
    bits = np.unpackbits(r["bitmask"].cpu().numpy(), axis=1, bitorder="little")[:, : kb * kb].reshape(2, kb, kb).astype(bool)
    for h in range(2):
        idxs = [po.perm_index(*grid, text, t) for t in range(6)]
        ref = pc.calibrate_head(q[0, h].float().numpy(), k[0, h].float().numpy(), idxs, block, EPS, SIGMA, ALPHA, DENSITY, k_img, REL)
        for t in range(6):
            assert mq[t, h] == pytest.approx(ref["orders"][t]["m_quant"], rel=2 * REL)
        chosen = ref["orders"][int(r["h_perm_ids"][h])]
        assert np.allclose(bsum[h], chosen["sum"], rtol=REL, atol=1e-30)
        # the mask is the oracle's rule on the kernel's sums, and on the exact sums but for blocks that tie within REL
        assert np.array_equal(bits[h], pc.mask_from_block_sums(bsum[h].astype(np.float64), float(np.float32(DENSITY)), k_img))
        want = pc.mask_from_block_sums(chosen["sum"], float(np.float32(DENSITY)), k_img)
        worst_live = chosen["sum"][:k_img, :k_img][want[:k_img, :k_img]].min()
        differ = bits[h] != want
        assert np.all(np.abs(chosen["sum"][differ] / worst_live - 1.0) <= 2 * REL)

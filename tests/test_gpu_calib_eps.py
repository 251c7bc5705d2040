"""Calibration statistics over the whole range of eps that the entry points take: sums and maxima do not depend on it, and
the count follows it where it leaves the range in which it scales the exponent (2^-100 .. 1)."""
import numpy as np
import pytest

from oracle import paro_calibration as pc

pytestmark = pytest.mark.gpu

TIE = 2e-4  # as in the calibration parity tests: fp32 sums, logits of some 100 octaves, hardware exp2
EDGE = float(np.float32(2.0 ** -100))
EPS = [1e-45, 1e-40, 1e-37, float(np.nextafter(np.float32(EDGE), np.float32(0))), EDGE, 1e-3, 1.0, float(np.nextafter(np.float32(1), np.float32(2))), 3.0, 1e10, 3e38,
       float("inf")]


@pytest.mark.parametrize("block,d,grid", [(64, 64, (3, 5, 7)), (64, 128, (5, 9, 8)), (32, 64, (3, 5, 7)), (32, 128, (2, 9, 15))])
@pytest.mark.parametrize("gain", [1.0, 8.0])  # all of P above 1e-5; P down to 1e-68, a third of it below 2^-100
def test_statistics_for_every_eps(block, d, grid, gain):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(1, 1, d, *grid, 0, block)
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    gen = torch.Generator().manual_seed(n + d)
    q, k = (torch.randn((1, 1, n, d), generator=gen) for _ in range(2))
    q, k = (gain * q).to(torch.bfloat16), (gain ** 0.5 * k).to(torch.bfloat16)
    p = pc.attention_map(q[0, 0].float().numpy(), k[0, 0].float().numpy())
    assert (p.min() > 1e-6) if gain == 1.0 else (p.min() < 1e-33)
    z = dict(device="cuda:0")
    ids = np.zeros(1, np.uint8)
    q16, k16 = (torch.empty(pb.codes_shape(s, 16, pb.PARO_ROWS), dtype=torch.bfloat16, **z) for _ in range(2))
    sc = torch.empty((1, 1, kb), dtype=torch.float32, **z)
    pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, q.to("cuda:0"), q16, sc)
    pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, k.to("cuda:0"), k16, sc)
    rows = torch.zeros((pb.paro_calib_row_stats_bytes(s),), dtype=torch.uint8, **z)
    pb.paro_calib_row_stats(s, q16, k16, rows)
    for eps in EPS:
        if gain > 1.0 and eps < 1e-33:
            continue  # P below the smallest normal binary32 is zero in the kernel, not in the map
        ref = pc.block_stats(p, block, float(np.float32(eps)), TIE)
        for form in ("one call", "from rows"):
            out = [torch.full((1, 1, kb, kb), -1, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
            if form == "one call":
                pb.paro_calib_block_stats(s, q16, k16, eps, *out)
            else:
                pb.paro_calib_block_stats_from_rows(s, ids, q16, k16, rows, eps, *out)
            bsum, bmax, bcnt = (x[0, 0].cpu().numpy() for x in out)
            assert np.allclose(bsum, ref["sum"], rtol=TIE, atol=1e-30), (form, eps)
            assert np.allclose(bmax, ref["max"], rtol=TIE, atol=1e-30), (form, eps)
            assert np.all(bcnt >= ref["cnt_lo"]) and np.all(bcnt <= ref["cnt_hi"]), (form, eps)


@pytest.mark.parametrize("eps", [0.0, -1.0, float("nan")])
def test_refused(eps):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(1, 1, 64, 1, 8, 8, 0, 64)
    z = dict(device="cuda:0")
    x = torch.zeros(pb.codes_shape(s, 16, pb.PARO_ROWS), dtype=torch.bfloat16, **z)
    out = [torch.zeros((1, 1, 1, 1), dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
    rows = torch.zeros((pb.paro_calib_row_stats_bytes(s),), dtype=torch.uint8, **z)
    with pytest.raises(pb.ParoError):
        pb.paro_calib_block_stats(s, x, x, eps, *out)
    with pytest.raises(pb.ParoError):
        pb.paro_calib_block_stats_from_rows(s, np.zeros(1, np.uint8), x, x, rows, eps, *out)

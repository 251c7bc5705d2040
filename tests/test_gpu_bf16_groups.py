"""bf16 mode, block 64: a lane holds one query of each of several groups of 16, and one look at the sum of their exponentials decides
whether references have to move.  A query that is NaN must not hide that another query of the same lane climbs, and must not make the others
move either."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bad,climbs", [(5, 21), (21, 5), (5, 37), (53, 5), (60, 44), (None, 21)])
def test_nan_query_does_not_hide_a_climb(d, bad, climbs):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd import workloads as wl
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 1, d, 1, 16, 9, 0, 64)  # 144 tokens: two whole blocks and one of 16
    n = pb.paro_ntokens(s)
    pa = ParoAttention(s, [0], wl.pack_bitmask(np.ones((1, 3, 3), np.uint8)), 16, 16, torch.float32)
    gen = torch.Generator().manual_seed(d)
    q, k, v = (torch.randn((n, d), generator=gen).bfloat16() for _ in range(3))
    u = torch.sign(torch.randn((d,), generator=gen)).bfloat16()
    q[climbs] = 4 * u
    k[100:104] += 8 * u  # logits of about 4 * 8 * sqrt(d) * log2(e): 369 and 522 octaves above those of the first block
    if bad is not None:
        q[bad] = float("nan")
    pa.prepare_fused_qkv(*(x.float()[None, None].contiguous().cuda() for x in (q, k, v)))
    o = pa.attend_fused()[0, 0].double().cpu()
    ref = torch.softmax(q.double() @ k.double().T / np.sqrt(d), -1) @ v.double()
    rows = [i for i in range(n) if i != bad]
    # P is rounded to bf16 (2^-9 of each term) and the logits to fp32: under 1 % of the row's largest value
    assert torch.isfinite(o[rows]).all()
    assert float((o[rows] - ref[rows]).abs().max()) <= 1e-2 * float(v.double().abs().max())
    if bad is not None:
        assert torch.isnan(o[bad]).all()


@pytest.mark.parametrize("d", [64, 128])
def test_nan_query_does_not_move_the_other_references(d):
    """References move where a block's sum passes 2^64, and nothing less: rows that climb by some 20 octaves keep theirs, whatever
    the other queries of their wavefront hold, so their bits are the same beside a query of zeros and beside one of NaN."""
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd import workloads as wl
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 1, d, 1, 16, 21, 0, 64)  # 336 tokens: five whole blocks and one of 16
    n = pb.paro_ntokens(s)
    pa = ParoAttention(s, [0], wl.pack_bitmask(np.ones((1, 6, 6), np.uint8)), 16, 16, torch.float32)
    gen = torch.Generator().manual_seed(d)
    q, k, v = (torch.randn((n, d), generator=gen) for _ in range(3))
    u = torch.sign(torch.randn((d,), generator=gen))
    q += 0.5 * u
    for b in range(1, 6):
        k[64 * b :] += u  # logits of a block lie about 0.5 * sqrt(d) * log2(e), 6 and 8 octaves, above those of the one before
    bad = [5, 70, 149, 250, 330]

    def layer(value):
        q[bad] = value
        pa.prepare_fused_qkv(*(x[None, None].contiguous().cuda() for x in (q, k, v)))
        return pa.attend_fused()[0, 0].cpu()

    rows = [i for i in range(n) if i not in bad]
    zero, nan = layer(0.0), layer(float("nan"))
    assert torch.isfinite(zero).all() and torch.isnan(nan[bad]).all()
    assert torch.equal(nan[rows], zero[rows])

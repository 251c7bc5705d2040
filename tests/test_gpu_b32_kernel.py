"""The integer kernel of block 32 runs the products of a block beside the exponentials of its neighbours: checked against the oracle
where the order of things changes - rows of none to three blocks, on either side of eight and sixteen blocks and of the chunks of 64
column indices, the ragged block alone and behind others, padded query rows - and with V scales of very different and of very
large and small size (each row by itself: test_gpu_v_scale_spread.py)."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2506_16054_amd import workloads as wl
from tests.helpers import check_attention, oracle_head

pytestmark = pytest.mark.gpu

GRID = (1, 11, 381)  # 4191 tokens: 130 blocks of 32 and one of 31
LENGTHS = {0: 0, 1: 1, 2: 2, 3: 3, 4: 7, 5: 8, 6: 9, 7: 15, 8: 16, 9: 17, 10: 63, 11: 64, 12: 65, 13: 66, 14: 127, 15: 129, 16: 130}
ONLY_LAST, ALL, EVERY_OTHER, LAST_ROW = 30, 40, 41, 130


def _run(d, bits, grid, masks, q, k, v, rows, block_gain=None):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 1, d, *grid, 0, 32)
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    q, k, v = (x.astype(np.float32) for x in (q, k, v))
    pa = ParoAttention(s, np.zeros(1, np.uint8), wl.pack_bitmask(masks), *bits, torch.float32)
    dev = [torch.from_numpy(x).reshape(1, 1, n, d).to("cuda:0") for x in (q, k, v)]
    pa.o.fill_(float("nan"))
    got = pa.run_fused(*dev).clone()
    pa.op.fill_(float("nan"))
    assert torch.equal(pa.run(*dev), got)
    assert bool((pa.op[0, 0, n:] == 0).all())
    w = SimpleNamespace(F=grid[0], Hg=grid[1], Wg=grid[2], T_text=0, N=n, npad=32 * kb, block=32, d=d, bits_qk=bits[0], bits_pv=bits[1])
    ref = oracle_head(w, q, k, v, 0, pa.h_row_ptr[0], pa.h_col_idx, row_blocks=rows)
    o = got.cpu().numpy()[0, 0].astype(np.float64)
    assert np.isfinite(o).all()
    for i in rows:  # (the bar's element-wise bound is for values of the order of V's, so a row's largest V factor comes off first)
        at = np.arange(32 * i, min(32 * i + 32, n))
        g = 1.0 if block_gain is None else float(np.max(block_gain[masks[0, i]], initial=1e-300))
        if masks[0, i].any():
            check_attention(o[at] / g, ref["o"][at] / g, ref["flip_risk"][at] / g, 2e-2, 1e-2)
        else:
            assert not o[at].any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bits", [(8, 8), (8, 4), (4, 8), (4, 4)])
def test_row_lengths_chunks_and_ragged_blocks(d, bits):
    rng = np.random.default_rng(d + sum(bits))
    masks = np.zeros((1, 131, 131), bool)
    for i, count in LENGTHS.items():
        masks[0, i, rng.choice(130, count, replace=False)] = True
    masks[0, ALL] = masks[0, LAST_ROW] = True
    masks[0, EVERY_OTHER, ::2] = True
    masks[0, ONLY_LAST, 130] = True
    q, k, v = (rng.standard_normal((4191, d)) for _ in range(3))
    _run(d, bits, GRID, masks, q, k, v, sorted(LENGTHS) + [ONLY_LAST, ALL, EVERY_OTHER, LAST_ROW])


# log2 of the factors on the blocks of V (the ragged one last): equal; far apart; very large and very small
@pytest.mark.parametrize("d,bits", [(64, (8, 8)), (128, (8, 8)), (64, (4, 8)), (64, (8, 4))])
@pytest.mark.parametrize("gains", [(0, 0, 0, 0, 0), (0, -26, -13, 0, -26), (-30, 0, -15, 0, -2), (98, 98, 98, 90, 98), (110, 110, 110, 105, 110),
                                   (-53, -53, -53, -60, -53), (-57, -57, -57, -57, -57), (-90, -90, -90, -90, -90), (40, -40, 0, 20, -20)])
def test_v_scales_of_a_row_in_and_out_of_range(d, bits, gains):
    rng = np.random.default_rng(3)
    q, k, v = (rng.standard_normal((150, d)) for _ in range(3))
    masks = np.ones((1, 5, 5), bool)
    masks[0, 2, 1::2] = False
    gain = 2.0 ** np.array(gains, np.float64)
    _run(d, bits, (1, 10, 15), masks, q, k, v * np.repeat(gain, 32)[:150, None], list(range(5)), gain)


@pytest.mark.parametrize("d", [64, 128])
def test_row_maximum_climbing_hundreds_of_octaves(d):
    rng = np.random.default_rng(5)
    q, k, v = (rng.standard_normal((640, d)) for _ in range(3))
    q, k = 3.0 * np.abs(q), np.abs(k) * np.linspace(0.05, 9.0, 640)[:, None]
    logit = q[:1] @ k.T / np.sqrt(d) * np.log2(np.e)
    assert logit.max() - logit.min() > 200
    _run(d, (8, 8), (1, 20, 32), np.ones((1, 20, 20), bool), q, k, v, list(range(20)))

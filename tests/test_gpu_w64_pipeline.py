"""The integer kernels of d = 64, block 64 run the products of a block beside the exponentials of its neighbours: checked
against the oracle where the order of things changes - rows of none to three blocks, odd and even numbers of blocks, lists
that end around a chunk of 64 column indices, the ragged last block alone and behind others, padded query rows - in each of the
three ways the exponent is formed: folded (8-bit P codes, ordinary scales), scaled (4-bit P codes) and exact (scales beyond
the range of the other two)."""
from types import SimpleNamespace

import numpy as np
import pytest

from tests.helpers import check_attention, oracle_head
from paper_2506_16054_amd import workloads as wl

pytestmark = pytest.mark.gpu

LENGTHS = {0: 0, 1: 1, 2: 2, 3: 3, 7: 62, 8: 63, 9: 64, 10: 65, 11: 66, 20: 127, 21: 128, 22: 129, 23: 130}  # row block: live blocks
ONLY_LAST, LAST_ROW = 30, 130  # a row with the ragged column block alone; the ragged row block


def _run(grid, masks, q, k, v, bits_qk, bits_pv, rows, gain_qk=1.0, gain_v=1.0, raw_q=False, rel=1e-2, max_abs=2e-2):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 1, 64, *grid, 0, 64)
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    q, k, v = (np.float32(g) * x.astype(np.float32) for g, x in ((gain_qk, q), (gain_qk, k), (gain_v, v)))
    pa = ParoAttention(s, np.zeros(1, np.uint8), wl.pack_bitmask(masks), bits_qk, bits_pv, torch.float32)
    dev = [torch.from_numpy(x).reshape(1, 1, n, 64).to("cuda:0") for x in (q, k, v)]
    pa.o.fill_(float("nan"))
    got = pa.run_fused(*dev).clone()
    pa.op.fill_(float("nan"))
    assert torch.equal(pa.run(*dev), got)  # the padded form, and the inverse reorder as a call of its own
    assert bool((pa.op[0, 0, n:] == 0).all())
    if raw_q:
        assert torch.equal(pa.run_rawq(*dev), got)
    w = SimpleNamespace(F=grid[0], Hg=grid[1], Wg=grid[2], T_text=0, N=n, npad=64 * kb, block=64, d=64, bits_qk=bits_qk, bits_pv=bits_pv)
    ref = oracle_head(w, q, k, v, 0, pa.h_row_ptr[0], pa.h_col_idx, row_blocks=rows)
    at = np.concatenate([np.arange(64 * i, min(64 * i + 64, n)) for i in rows])
    o = got.cpu().numpy()[0, 0].astype(np.float64)
    assert np.isfinite(o).all()
    # (the bar's element-wise bound is for values of the order of V's, so V's factor comes off first)
    check_attention(o[at] / gain_v, ref["o"][at] / gain_v, ref["flip_risk"][at] / gain_v, max_abs, rel)


def _masks():
    masks = np.zeros((1, 131, 131), bool)
    rng = np.random.default_rng(131)
    for i, count in LENGTHS.items():
        masks[0, i, rng.choice(130, count, replace=False)] = True  # without the ragged column block
    masks[0, 40] = masks[0, LAST_ROW] = True
    masks[0, 41, ::2] = True  # ends with it: 66 blocks
    masks[0, ONLY_LAST, 130] = True
    return masks


@pytest.mark.parametrize("bits", [(8, 8), (8, 4), (4, 8), (4, 4)])
def test_row_lengths_chunks_and_ragged_blocks(bits):
    grid = (1, 67, 125)  # 8375 tokens: 130 blocks of 64 and one of 55
    rng = np.random.default_rng(sum(bits))
    q, k, v = (rng.standard_normal((8375, 64)) for _ in range(3))
    rows = sorted(LENGTHS) + [ONLY_LAST, 40, 41, LAST_ROW]
    _run(grid, _masks(), q, k, v, *bits, rows, raw_q=bits[0] == 8)


@pytest.mark.parametrize("bits", [(8, 8), (8, 4), (4, 8), (4, 4)])
@pytest.mark.parametrize("gain_qk,gain_v", [(6.0, 1.0), (100.0, 2.0 ** -60), (2.0 ** -60, 2.0 ** 120), (1.0, 2.0 ** -100)])
def test_scales_past_the_folded_form_and_extreme_ones(bits, gain_qk, gain_v):
    """6, 100: logits of some hundred and of some 10^4 octaves, past the line of the folded form; 2^-60: all logits equal to within
    rounding; 2^120: beyond the line where the sums of P V are held smaller."""
    grid = (1, 10, 35)  # 350 tokens: 5 blocks of 64 and one of 30
    rng = np.random.default_rng(7)
    q, k, v = (rng.standard_normal((350, 64)) for _ in range(3))
    masks = np.ones((1, 6, 6), bool)
    masks[0, 2, 1::2] = False
    _run(grid, masks, q, k, v, *bits, list(range(6)), gain_qk, gain_v, raw_q=bits[0] == 8)


@pytest.mark.parametrize("bits", [(8, 8), (8, 4), (4, 8), (4, 4)])
@pytest.mark.parametrize("octave", [89, 91, 101])
def test_exact_form_beyond_the_scaled_one(bits, octave):
    """Logit scales of 1.4 * 2^octave per integer step: below and above 2^90, where the scaled form gives way to the exact one
    (8-bit P codes take the exact form at all three).  A row of Q and a row of K have one channel that counts, of opposite signs, so
    logits are 0 or of -2^100 octaves and every maximum is 0: attention is the mean of V over the keys of other channels.  (The offset of
    an exponent holds minus the maximum and log2 of the largest code in one float, so maxima this large are out of range.)"""
    grid = (1, 10, 35)
    rng = np.random.default_rng(11)
    one, top = (64.0, 127.0) if bits[0] == 8 else (4.0, 7.0)
    q, k = np.zeros((2, 350, 64))
    for x, own, sign in ((q, 63, 1.0), (k, 62, -1.0)):
        x[range(350), rng.integers(0, 4, 350)] = one * sign
        x[:, own] = top  # the largest value of every block, in a channel that the other tensor leaves at 0
    masks = np.ones((1, 6, 6), bool)
    masks[0, 2, 1::2] = False
    # scale per step: gain^2 * log2(e) / 8, of 4-bit codes (times 16 each) / 256
    gain = 2.0 ** ((octave + 3) // 2 + (0 if bits[0] == 8 else 4))
    c = gain * gain * 1.4426950408889634 / 8 / (1 if bits[0] == 8 else 256)
    assert (c < 2.0**90) == (octave == 89) and 1.4 < c / 2.0**octave < 1.5
    _run(grid, masks, q, k, rng.standard_normal((350, 64)), *bits, list(range(6)), gain, raw_q=bits[0] == 8)

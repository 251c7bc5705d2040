"""The kernel with four wavefronts of 16 queries per row block (block 64; d = 128, and d = 64 up to 1536 row blocks) multiplies K Q of a
block while it exponentiates the one before and brings tiles in two blocks ahead: checked against the oracle where the order of
things changes - rows of none to nine blocks and around chunks of 64 column indices, the ragged block alone and behind others, padded
query rows - in every combination of bits, with Q quantized in the kernel too, with V scales of very different size (each row by
itself: test_gpu_v_scale_spread.py), and on either side of the numbers of row blocks at which d = 64 changes kernels."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2506_16054_amd import workloads as wl
from tests.helpers import check_attention, oracle_head

pytestmark = pytest.mark.gpu

GRID = (1, 79, 106)  # 8374 tokens: 130 blocks of 64 and one of 54
LENGTHS = {0: 0, 1: 1, 2: 2, 3: 3, 4: 4, 5: 5, 6: 8, 7: 9, 8: 62, 9: 63, 10: 64, 11: 65, 12: 66, 13: 67, 14: 127, 15: 129, 16: 130}
ONLY_LAST, ALL, LAST_ROW = 30, 40, 130
BITS = [(8, 8), (8, 4), (4, 8), (4, 4)]


def _run(d, bits, grid, masks, q, k, v, rows, block_gain=None, heads=1):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, heads, d, *grid, 0, 64)
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    q, k, v = (x.astype(np.float32) for x in (q, k, v))
    pa = ParoAttention(s, np.zeros(heads, np.uint8), wl.pack_bitmask(np.repeat(masks, heads, axis=0)), *bits, torch.float32)
    dev = [torch.from_numpy(x).reshape(1, 1, n, d).to("cuda:0").repeat(1, heads, 1, 1) for x in (q, k, v)]
    pa.o.fill_(float("nan"))
    got = pa.run_fused(*dev).clone()
    pa.op.fill_(float("nan"))
    assert torch.equal(pa.run(*dev), got)
    assert bool((pa.op[:, :, n:] == 0).all())
    if bits[0] == 8:
        assert torch.equal(pa.run_rawq(*dev), got)
    assert torch.equal(got, got[:, :1].expand_as(got))
    w = SimpleNamespace(F=grid[0], Hg=grid[1], Wg=grid[2], T_text=0, N=n, npad=64 * kb, block=64, d=d, bits_qk=bits[0], bits_pv=bits[1])
    ref = oracle_head(w, q, k, v, 0, pa.h_row_ptr[0], pa.h_col_idx, row_blocks=rows)
    o = got.cpu().numpy()[0, 0].astype(np.float64)
    assert np.isfinite(o).all()
    for i in rows:  # (the bar's element-wise bound is for values of the order of V's, so a row's largest V factor comes off first)
        at = np.arange(64 * i, min(64 * i + 64, n))
        g = 1.0 if block_gain is None else float(np.max(block_gain[masks[0, i]], initial=1e-300))
        if masks[0, i].any() and bits[1] == 8:
            check_attention(o[at] / g, ref["o"][at] / g, ref["flip_risk"][at] / g, 2e-2, 1e-2)
        elif masks[0, i].any():
            # One 4-bit P code at a rounding tie moves the d elements of its query by up to a seventh of its term, and a row of one block has
            # few terms: here the bound is every element's own tie allowance beside the relative error, not a share of the tensor.
            diff = np.abs(o[at] - ref["o"][at])
            assert np.linalg.norm(diff) <= 1e-2 * np.linalg.norm(ref["o"][at])
            assert np.all(diff / g <= 2e-2 + ref["flip_risk"][at] / g)
        else:
            assert not o[at].any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bits", BITS)
def test_row_lengths_chunks_and_ragged_blocks(d, bits):
    rng = np.random.default_rng(d + sum(bits))
    masks = np.zeros((1, 131, 131), bool)
    for i, count in LENGTHS.items():
        masks[0, i, rng.choice(130, count, replace=False)] = True
    masks[0, ALL] = masks[0, LAST_ROW] = True
    masks[0, ONLY_LAST, 130] = True
    q, k, v = (rng.standard_normal((8374, d)) for _ in range(3))
    _run(d, bits, GRID, masks, q, k, v, sorted(LENGTHS) + [ONLY_LAST, ALL, LAST_ROW])


# log2 of the factors on the blocks of V (the ragged one last), as for block 32
@pytest.mark.parametrize("d,bits", [(64, (8, 8)), (128, (8, 8)), (128, (4, 8)), (128, (8, 4))])
@pytest.mark.parametrize("gains", [(0, -26, -13, 0, -26), (-30, 0, -15, 0, -2), (98, 98, 98, 90, 98), (110, 110, 110, 105, 110),
                                   (-53, -53, -53, -60, -53), (-57, -57, -57, -57, -57), (-90, -90, -90, -90, -90)])
def test_v_scales_of_a_row_in_and_out_of_range(d, bits, gains):
    rng = np.random.default_rng(3)
    q, k, v = (rng.standard_normal((280, d)) for _ in range(3))
    masks = np.ones((1, 5, 5), bool)
    masks[0, 2, 1::2] = False
    gain = 2.0 ** np.array(gains, np.float64)
    _run(d, bits, (1, 10, 28), masks, q, k, v * np.repeat(gain, 64)[:280, None], list(range(5)), gain)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bits", [(8, 8), (8, 4)])
def test_row_maximum_climbing_hundreds_of_octaves(d, bits):
    rng = np.random.default_rng(5)
    q, k, v = (rng.standard_normal((640, d)) for _ in range(3))
    q, k = 3.0 * np.abs(q), np.abs(k) * np.linspace(0.05, 9.0, 640)[:, None]
    logit = q[:1] @ k.T / np.sqrt(d) * np.log2(np.e)
    assert logit.max() - logit.min() > 200
    _run(d, bits, (1, 20, 32), np.ones((1, 10, 10), bool), q, k, v, list(range(10)))


# heads x row blocks on either side of 1536 in all; of 1280 and 1024, where rows of fewer than 8 blocks change kernels (7.5 of 8 are live)
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("heads,blocks", [(192, 8), (193, 8), (160, 8), (161, 8), (128, 8), (129, 8), (128, 12), (129, 12)])
def test_both_sides_of_the_number_of_row_blocks_at_which_the_kernel_changes(bits, heads, blocks):
    rng = np.random.default_rng(heads)
    n = 64 * blocks - 12
    q, k, v = (rng.standard_normal((n, 64)) for _ in range(3))
    masks = np.ones((1, blocks, blocks), bool)
    masks[0, 3, 1::2] = False
    _run(64, bits, (1, n // 4, 4), masks, q, k, v, list(range(blocks)), heads=heads)

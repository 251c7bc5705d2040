"""Calibration in two steps (row statistics once, block statistics per axis order) against the one-call form, and
the mask selection at the sizes where the kernels change: keys per thread, registers or memory, ties.  The two forms add a
row's denominator in another order, in binary64: they are equal bit for bit unless a sum lies within its own rounding error
of a binary32 rounding boundary, which none of these inputs' (fixed) sums do."""
import numpy as np
import pytest

from oracle import paro_calibration as pc
from oracle import paro_oracle as po
from paper_2506_16054_amd import workloads as wl

pytestmark = pytest.mark.gpu


# row blocks: fewer than one group of four, a whole group, a group and a ragged block; more than one column chunk
@pytest.mark.parametrize("block,d,grid", [(64, 64, (1, 5, 9)), (64, 64, (4, 8, 8)), (64, 128, (3, 9, 11)), (32, 64, (2, 9, 15)),
                                          (32, 128, (1, 8, 16)), (64, 64, (3, 20, 19))])
def test_block_statistics_from_rows_equal_the_one_call_form(block, d, grid):
    import torch

    from paper_2506_16054_amd import binding as pb

    F, Hg, Wg = grid
    s = pb.make_shape(2, 3, d, F, Hg, Wg, 0, block)
    k = pb.paro_nblocks(s)
    gen = torch.Generator(device="cuda:0").manual_seed(block + d + Hg)
    x, y = (torch.randn((2, 3, pb.paro_ntokens(s), d), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    z = dict(device="cuda:0")
    q16, k16 = (torch.empty(pb.codes_shape(s, 16, pb.PARO_ROWS), dtype=torch.bfloat16, **z) for _ in range(2))
    sc = torch.empty((2, 3, k), dtype=torch.float32, **z)
    rows = torch.zeros((pb.paro_calib_row_stats_bytes(s),), dtype=torch.uint8, **z)
    shape = (2, 3, k, k)
    for ids in ([0, 0, 0], [1, 5, 3]):
        ids = np.array(ids, np.uint8)
        pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, x, q16, sc)
        pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, y, k16, sc)
        if not ids.any():
            pb.paro_calib_row_stats(s, q16, k16, rows)
        one = [torch.full(shape, -1, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
        two = [torch.full(shape, -2, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
        pb.paro_calib_block_stats(s, q16, k16, 2e-3, *one)
        pb.paro_calib_block_stats_from_rows(s, ids, q16, k16, rows, 2e-3, *two)
        for a, b in zip(one, two):
            assert torch.equal(a, b)
        # and against the float64 map of one head: fp32 sums of products of bf16 values
        h = 1
        idx = po.perm_index(F, Hg, Wg, 0, int(ids[h]))
        ref = pc.block_stats(pc.reorder_map(pc.attention_map(x[1, h].float().cpu().numpy(), y[1, h].float().cpu().numpy()), idx), block, 2e-3, 2e-4)
        assert np.allclose(two[0][1, h].cpu().numpy(), ref["sum"], rtol=2e-4, atol=1e-30)
        assert np.allclose(two[1][1, h].cpu().numpy(), ref["max"], rtol=2e-4, atol=1e-30)
        cnt = two[2][1, h].cpu().numpy()
        assert np.all(cnt >= ref["cnt_lo"]) and np.all(cnt <= ref["cnt_hi"])


# 8 and 80 keys per thread of a 1024-thread workgroup end at 90 x 90 and 286 x 286 blocks
@pytest.mark.parametrize("k", [1, 3, 32, 90, 91, 286, 287])
@pytest.mark.parametrize("values", [3, 0])
def test_mask_selection_at_the_kernels_size_limits(k, values):
    """values 3: three distinct sums, so that the threshold falls among many equal ones; 0: all different, wide range."""
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(2, 2, 64, 1, k, 32, 0, 32)
    rng = np.random.default_rng(k)
    sums = rng.integers(0, values, size=(2, 2, k, k)) * 0.5 if values else np.exp(rng.uniform(-30, 5, size=(2, 2, k, k)))
    sums = sums.astype(np.float32)
    d_sums = torch.from_numpy(sums).to("cuda:0")
    for density in (0.0, 0.3, 0.55, 1.0):
        bits = torch.full((2, (k * k + 7) // 8), 255, dtype=torch.uint8, device="cuda:0")
        pb.paro_calib_mask(s, d_sums, density, bits)
        got = np.unpackbits(bits.cpu().numpy(), axis=1, bitorder="little")
        assert not got[:, k * k:].any()
        for h in range(2):
            want = pc.mask_from_block_sums((sums[0, h] + sums[1, h]).astype(np.float64), float(np.float32(density)), k)
            assert np.array_equal(got[h, : k * k].reshape(k, k).astype(bool), want), (density, h)


def test_pick_takes_every_heads_own_order():
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(2, 5, 64, 1, 3, 32, 0, 32)
    six = torch.arange(6 * 2 * 5 * 9, dtype=torch.float32, device="cuda:0").view(6, 2, 5, 3, 3)
    ids = torch.tensor([5, 0, 3, 1, 4], dtype=torch.uint8, device="cuda:0")
    out = torch.empty((2, 5, 3, 3), dtype=torch.float32, device="cuda:0")
    pb.paro_calib_pick(s, six, ids, out)
    assert torch.equal(out, torch.stack([six[int(ids[h]), :, h] for h in range(5)], dim=1))


# heads of one to three row blocks on either side of the number of workgroups at which the one-call form changes
@pytest.mark.parametrize("block,d,heads,n", [(64, 64, 768, 130), (64, 64, 769, 130), (64, 128, 256, 77), (64, 128, 257, 77), (32, 64, 256, 90),
                                             (32, 64, 257, 90), (32, 128, 256, 33), (32, 128, 257, 33)])
def test_both_forms_of_the_one_call_form(block, d, heads, n):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(heads, 1, d, 1, 1, n, 0, block)
    k = pb.paro_nblocks(s)
    gen = torch.Generator(device="cuda:0").manual_seed(heads + n)
    x, y = (torch.randn((heads, 1, n, d), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    z = dict(device="cuda:0")
    ids = np.zeros(1, np.uint8)
    q16, k16 = (torch.empty(pb.codes_shape(s, 16, pb.PARO_ROWS), dtype=torch.bfloat16, **z) for _ in range(2))
    sc = torch.empty((heads, 1, k), dtype=torch.float32, **z)
    pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, x, q16, sc)
    pb.paro_permute_quantize(s, 16, pb.PARO_ROWS, ids, y, k16, sc)
    rows = torch.zeros((pb.paro_calib_row_stats_bytes(s),), dtype=torch.uint8, **z)
    pb.paro_calib_row_stats(s, q16, k16, rows)
    one = [torch.full((heads, 1, k, k), -1, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
    two = [torch.full((heads, 1, k, k), -2, dtype=t, **z) for t in (torch.float32, torch.float32, torch.int32)]
    pb.paro_calib_block_stats(s, q16, k16, 2e-3, *one)
    pb.paro_calib_block_stats_from_rows(s, ids, q16, k16, rows, 2e-3, *two)
    for a, b in zip(one, two):
        assert torch.equal(a, b)
    for h in (0, heads // 2, heads - 1):
        ref = pc.block_stats(pc.attention_map(x[h, 0].float().cpu().numpy(), y[h, 0].float().cpu().numpy()), block, 2e-3, 2e-4)
        assert np.allclose(one[0][h, 0].cpu().numpy(), ref["sum"], rtol=2e-4, atol=1e-30)
        assert np.allclose(one[1][h, 0].cpu().numpy(), ref["max"], rtol=2e-4, atol=1e-30)
        cnt = one[2][h, 0].cpu().numpy()
        assert np.all(cnt >= ref["cnt_lo"]) and np.all(cnt <= ref["cnt_hi"])

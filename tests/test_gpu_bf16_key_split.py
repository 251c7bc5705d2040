"""The bf16 kernels of block 64, whose wavefronts split the keys of every block, where that can go wrong: a ragged last
block that leaves the upper wavefronts without keys (alone in a row, last of several), rows of none, one, two and three
blocks, more than 64 blocks, and rows whose logits climb past the reference by less and by more than the exponential's
range, at the first block of a row and later, in the keys of either wavefront."""
import numpy as np
import pytest

from paper_2506_16054_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _check(d, n_grid, masks, q, k, v, dtype="f32"):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 1, d, *n_grid, 0, 64)
    n = pb.paro_ntokens(s)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    pa = ParoAttention(s, np.zeros(1, np.uint8), wl.pack_bitmask(masks), 16, 16, tdt)
    dev = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).to(tdt).reshape(1, 1, n, d).to("cuda:0") for x in (q, k, v)]
    pa.o.fill_(float("nan"))
    got_steps = pa.run(*dev).clone()
    got = pa.run_fused(*dev)
    assert torch.equal(got, got_steps)
    q64, k64, v64 = (x.double().cpu()[0, 0] for x in dev)
    live = torch.from_numpy(np.repeat(np.repeat(masks[0], 64, 0), 64, 1)[:n, :n])
    x = (q64 @ k64.T / d ** 0.5).masked_fill(~live, -float("inf"))
    p = torch.where(live.any(1, keepdim=True), torch.softmax(x, 1), torch.zeros(()).double())
    want = p @ v64
    err = (got.double().cpu()[0, 0] - want).norm() / want.norm()
    # P enters the second product rounded to bf16 (at most 2^-9 of each term); a bf16 output is rounded once more
    bound = 2.0 ** -9 * (2.0 if dtype == "bf16" else 1.0) + 1e-4
    assert torch.isfinite(got).all() and float(err) <= bound, float(err)
    assert bool((got.cpu()[0, 0][~live.any(1)] == 0).all())


@pytest.mark.parametrize("d", [64, 128])
# 360 = 5 * 64 + 40 tokens; 321 = 5 * 64 + 1 and 352 = 5 * 64 + 32: no keys of the last block for the upper wavefronts
@pytest.mark.parametrize("grid", [(5, 8, 9), (1, 3, 107), (1, 11, 32)])
def test_short_rows_and_ragged_blocks(d, grid):
    rng = np.random.default_rng(d + grid[1])
    n = grid[0] * grid[1] * grid[2]
    masks = np.zeros((1, 6, 6), bool)
    masks[0, 0, [5]] = True
    masks[0, 1, [0, 5]] = True
    masks[0, 2, [1, 2, 4]] = True
    masks[0, 4, :] = True
    masks[0, 5, [0, 1, 2, 3]] = True
    q, k, v = (rng.standard_normal((n, d)) for _ in range(3))
    _check(d, grid, masks, 2 * q, k, v)
    _check(d, grid, masks, 2 * q, k, v, "bf16")


@pytest.mark.parametrize("d", [64, 128])
def test_more_than_one_chunk_of_the_column_list(d):
    rng = np.random.default_rng(d)
    masks = np.ones((1, 68, 68), bool)
    masks[0, 3, ::2] = False
    q, k, v = (rng.standard_normal((4350, d)) for _ in range(3))
    _check(d, (5, 29, 30), masks, q, k, v)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("upper", [False, True])
@pytest.mark.parametrize("gain", [6.0, 30.0, 300.0])  # climbs of tens, hundreds and thousands of octaves
def test_logits_that_climb_past_the_reference(d, upper, gain):
    rng = np.random.default_rng(int(gain) + d)
    n = 64 * 6
    q = np.abs(rng.standard_normal((n, d)))
    k = np.abs(rng.standard_normal((n, d))) * 0.05
    # one key of block 2 and one of block 4 stand out, in the half of the keys that one wavefront owns
    k[2 * 64 + 40 * upper + 3] *= gain
    k[4 * 64 + 40 * upper + 7] *= 3.0 * gain
    v = rng.standard_normal((n, d))
    _check(d, (6, 8, 8), np.ones((1, 6, 6), bool), q, k, v)

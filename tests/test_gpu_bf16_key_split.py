"""The bf16 kernels of block 64, whose wavefronts split the keys of every block, where that can go wrong: a ragged last
block that leaves the upper wavefronts without keys (alone in a row, last of several), rows of none, one, two and three
blocks, more than 64 blocks, rows whose logits climb past the reference (a wavefront's first maximum) by less than the 64
octaves at which it is moved, by more, and by more than the exponential's range, in the keys of either wavefront and in
a ragged last block, and rows whose first block holds the largest logits."""
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
@pytest.mark.parametrize("gain", [6.0, 30.0, 300.0])  # climbs of at most 12, of 20 to 58 and of 68 to 640 octaves
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


def _climbs(d, q, k, half):
    """[rows]: octaves from a wavefront's first maximum of a row (over its half of block 0) to its largest logit, every block live."""
    r = [_bf16(x) for x in (q, k)]
    x = (r[0] @ r[1].T) * (1.4426950408889634 / d ** 0.5)
    own = np.arange(len(k)) % 64 // 32 == half
    first = x[:, own & (np.arange(len(k)) < 64)].max(1)
    return x[:, own].max(1) - first


def _bf16(x):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).double().numpy()


def _key(d, octaves):
    """A key whose logits against queries of |N(0, 1)| are about so many octaves (their channels add up to about 0.8 d)."""
    return octaves * d ** 0.5 / (1.4426950408889634 * 0.798 * d)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("upper", [False, True])
@pytest.mark.parametrize("octaves,lo,hi", [(20.0, 5.0, 64.0), (95.0, 64.0, 128.0), (300.0, 192.0, 450.0)])
def test_climbs_of_a_stated_size(d, upper, octaves, lo, hi):
    rng = np.random.default_rng(int(octaves) + d)
    n = 64 * 6
    q = np.abs(rng.standard_normal((n, d)))
    q *= 0.798 * d / q.sum(1, keepdims=True)  # all rows climb alike
    k = np.abs(rng.standard_normal((n, d))) * 0.05
    # one key of block 2 stands out, in the half of the keys that one wavefront owns, and one of block 4 by as much again
    k[2 * 64 + 40 * upper + 3] = _key(d, octaves)
    c = _climbs(d, q, k, int(upper))
    assert lo < c.min() and c.max() < hi and _climbs(d, q, k, int(not upper)).max() < 5.0
    k[4 * 64 + 40 * upper + 7] = _key(d, 2.0 * octaves)
    v = rng.standard_normal((n, d))
    _check(d, (6, 8, 8), np.ones((1, 6, 6), bool), q, k, v)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("upper", [False, True])
def test_the_largest_logits_in_the_first_block(d, upper):
    rng = np.random.default_rng(d)
    n = 64 * 6
    q = np.abs(rng.standard_normal((n, d)))
    k = np.abs(rng.standard_normal((n, d))) * 0.05
    k[40 * upper + 5] = _key(d, 300.0)  # the wavefront of the other half keeps a reference some 300 octaves lower
    assert _climbs(d, q, k, int(upper)).max() == 0.0
    v = rng.standard_normal((n, d))
    _check(d, (6, 8, 8), np.ones((1, 6, 6), bool), q, k, v)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("upper,tail", [(False, 40), (True, 40), (False, 20)])
@pytest.mark.parametrize("octaves,lo,hi", [(95.0, 64.0, 128.0), (250.0, 160.0, 320.0)])
def test_a_climb_in_the_ragged_last_block(d, upper, tail, octaves, lo, hi):
    """All logits lie far below 0, what a padded key would give: one that is not masked where the logits are formed anew takes
    the whole row."""
    rng = np.random.default_rng(int(octaves) + tail + d)
    n = 64 * 5 + tail
    q = np.abs(rng.standard_normal((n, d)))
    q *= 0.798 * d / q.sum(1, keepdims=True)
    k = rng.standard_normal((n, d)) * 0.05 + _key(d, -500.0)
    k[5 * 64 + 32 * upper + 3] = _key(d, -500.0 + octaves)
    c = _climbs(d, q, k, int(upper))
    assert lo < c.min() and c.max() < hi
    v = rng.standard_normal((n, d))
    _check(d, (1, n // 4, 4), np.ones((1, 6, 6), bool), q, k, v)

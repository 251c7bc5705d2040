"""The bf16 kernel whose wavefronts have 32 queries and 32 keys of every block (block 32; block 64, d = 64 up to 768 row blocks) multiplies K Q
of a block beside the exponentials of the one before: checked where the order of things changes - rows of none to four blocks and around
the chunks of 64 column indices, the ragged block alone and behind others - with logits that climb past a reference by less than the 64
octaves at which it is moved, by more, and past the exponential's range, in the middle of a row and in the ragged last block, and on
either side of the number of row blocks at which d = 64, block 64 changes kernels."""
import numpy as np
import pytest

from paper_2506_16054_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _check(block, d, grid, masks, q, k, v, dtype="f32", heads=1):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, heads, d, *grid, 0, block)
    n = pb.paro_ntokens(s)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    pa = ParoAttention(s, np.zeros(heads, np.uint8), wl.pack_bitmask(np.repeat(masks, heads, axis=0)), 16, 16, tdt)
    dev = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).to(tdt).reshape(1, 1, n, d).to("cuda:0").repeat(1, heads, 1, 1)
           for x in (q, k, v)]
    pa.o.fill_(float("nan"))
    pa.op.fill_(float("nan"))
    got_steps = pa.run(*dev).clone()
    assert bool((pa.op[:, :, n:] == 0).all())
    got = pa.run_fused(*dev)
    assert torch.equal(got, got_steps) and torch.equal(got, got[:, :1].expand_as(got))
    q64, k64, v64 = (x.double().cpu()[0, 0] for x in dev)
    live = torch.from_numpy(np.repeat(np.repeat(masks[0], block, 0), block, 1)[:n, :n])
    x = (q64 @ k64.T / d ** 0.5).masked_fill(~live, -float("inf"))
    p = torch.where(live.any(1, keepdim=True), torch.softmax(x, 1), torch.zeros(()).double())
    want = p @ v64
    err = (got.double().cpu()[0, 0] - want).norm() / want.norm()
    # P enters the second product rounded to bf16 (at most 2^-9 of each term); a bf16 output is rounded once more
    bound = 2.0 ** -9 * (2.0 if dtype == "bf16" else 1.0) + 1e-4
    assert torch.isfinite(got).all() and float(err) <= bound, float(err)
    assert bool((got.cpu()[0, 0][~live.any(1)] == 0).all())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid", [(5, 8, 5), (1, 7, 23), (1, 11, 16)])  # last block of 8, 1 and 16 tokens, 6 to 7 blocks
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_short_rows_and_ragged_blocks(d, grid, dtype):
    rng = np.random.default_rng(d + grid[1])
    n = grid[0] * grid[1] * grid[2]
    kb = -(-n // 32)
    masks = np.zeros((1, kb, kb), bool)
    for i, cols in enumerate(([kb - 1], [0, kb - 1], [1, 2, 4], [], range(kb), [0, 1, 2, 3])):
        masks[0, i, list(cols)] = True
    masks[0, kb - 1, [1, kb - 1]] = True
    q, k, v = (rng.standard_normal((n, d)) for _ in range(3))
    _check(32, d, grid, masks, 2 * q, k, v, dtype)


@pytest.mark.parametrize("d", [64, 128])
def test_chunks_of_the_column_list(d):
    rng = np.random.default_rng(d)
    masks = np.zeros((1, 131, 131), bool)
    for i in range(131):
        masks[0, i, rng.choice(131, (61 + i % 9) if i % 2 else (125 + i % 7), replace=False)] = True
    q, k, v = (rng.standard_normal((4179, d)) for _ in range(3))
    _check(32, d, (7, 3, 199), masks, q, k, v)


def _key(d, octaves):
    """A key whose logits against queries of |N(0, 1)| are about so many octaves (their channels add up to about 0.8 d)."""
    return octaves * d ** 0.5 / (1.4426950408889634 * 0.798 * d)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("octaves", [20.0, 95.0, 300.0])
@pytest.mark.parametrize("tail", [0, 9])
def test_logits_that_climb_past_the_reference(d, octaves, tail):
    """One key of block 2 stands out by `octaves`, one of block 4 by as much again, and with a ragged block one of its keys once more."""
    rng = np.random.default_rng(int(octaves) + d)
    n = 32 * 6 + tail
    kb = 7 if tail else 6
    q = np.abs(rng.standard_normal((n, d)))
    q *= 0.798 * d / q.sum(1, keepdims=True)  # all rows climb alike
    k = np.abs(rng.standard_normal((n, d))) * 0.05 - _key(d, 1000.0)  # all far below 0, what a padded key would give
    for at, times in ((2 * 32 + 11, 1.0), (4 * 32 + 30, 2.0), (n - 1, 3.0)):
        k[at] += _key(d, times * octaves)
    _check(32, d, (1, 1, n), np.ones((1, kb, kb), bool), q, k, rng.standard_normal((n, d)))


@pytest.mark.parametrize("heads", [128, 129])
def test_both_sides_of_the_number_of_row_blocks_at_which_the_kernel_changes(heads):
    rng = np.random.default_rng(heads)
    masks = np.ones((1, 6, 6), bool)  # 768 and 774 row blocks
    masks[0, 3, 1::2] = False
    masks[0, 4] = False
    q = np.abs(rng.standard_normal((360, 64)))
    k = np.abs(rng.standard_normal((360, 64))) * 0.05
    k[2 * 64 + 43] *= 100.0
    k[350] *= 300.0
    _check(64, 64, (1, 10, 36), masks, q, k, rng.standard_normal((360, 64)), heads=heads)

"""V scales of very different size in one row of blocks: an all-zero block of V (its scale is 1, whatever the others are) and a block of V
that is 2^8 .. 2^26 times larger and that one query of the tile attends while the others have P codes of 0 there.  Such a block
contributes exactly 0 to those queries, so each query row is held to its own relative error, not to the largest V of the tile.  And V of
any size under row maxima that climb from block to block, which the weights of the sums carry together."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2506_16054_amd import workloads as wl
from tests.helpers import oracle_head

pytestmark = pytest.mark.gpu

# (block, d, heads): every integer kernel; twice 200 heads of 5 blocks are past the number of row blocks at which block 64, d = 64 changes kernels
SHAPES = [(32, 64, 1), (32, 128, 1), (64, 64, 1), (64, 128, 1), (64, 64, 200)]
BITS = [(8, 8), (8, 4), (4, 8), (4, 4)]
BLOCKS = 5


def _check(block, d, heads, bits, q, k, v):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import ParoAttention

    n = q.shape[0]
    batch = 2 if heads > 1 else 1
    s = pb.make_shape(batch, heads, d, 1, 1, n, 0, block)
    masks = np.ones((1, BLOCKS, BLOCKS), bool)
    masks[0, 3, 2] = False  # a row of an even number of blocks among those of an odd one
    pa = ParoAttention(s, np.zeros(heads, np.uint8), wl.pack_bitmask(np.repeat(masks, heads, axis=0)), *bits, torch.float32)
    q, k, v = (x.astype(np.float32) for x in (q, k, v))
    dev = [torch.from_numpy(x).reshape(1, 1, n, d).to("cuda:0").repeat(batch, heads, 1, 1) for x in (q, k, v)]
    got = pa.run_fused(*dev).clone()
    assert torch.equal(got, got[:1, :1].expand_as(got))
    if pa.can_fuse_q:
        assert torch.equal(pa.run_rawq(*dev), got)
    w = SimpleNamespace(F=1, Hg=1, Wg=n, T_text=0, N=n, npad=BLOCKS * block, block=block, d=d, bits_qk=bits[0], bits_pv=bits[1])
    ref = oracle_head(w, q, k, v, 0, pa.h_row_ptr[0], pa.h_col_idx)
    norm = lambda x: np.linalg.norm(x, axis=1)  # noqa: E731
    o, want, risk = got[0, 0].cpu().numpy().astype(np.float64), ref["o"], ref["flip_risk"][:n]
    assert np.isfinite(o).all()
    # row by row: 1e-3 (the largest that fp32 sums and the exponent's rounding at its bound, 2^-12 ln 2, leave of it is 3e-4) beside what P
    # codes at a rounding tie can move
    off = norm(o - want) - norm(risk)
    worst = int(np.argmax(off / norm(want)))
    assert (off <= 1e-3 * norm(want)).all(), "row %d is off by %.1e of its norm" % (worst, off[worst] / norm(want)[worst])


@pytest.mark.parametrize("block,d,heads", SHAPES)
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("size", [1.0, 1e-2, 1e-4])
def test_block_of_zeros(block, d, heads, bits, size):
    rng = np.random.default_rng(block + d)
    n = BLOCKS * block - 10
    q, k, v = (rng.standard_normal((n, d)) for _ in range(3))
    v *= size
    v[2 * block : 3 * block] = 0.0
    _check(block, d, heads, bits, q, k, v)


@pytest.mark.parametrize("block,d,heads", SHAPES)
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("octaves", [8, 14, 20, 26])
def test_large_block_that_one_query_attends(block, d, heads, bits, octaves):
    rng = np.random.default_rng(octaves)
    n = BLOCKS * block - 10
    q, k, v = (rng.standard_normal((n, d)) for _ in range(3))
    # 16 channels decide who attends block 1, by a logit of +- 30 nats there and 0 elsewhere (one channel alone would make scales that take
    # another form of the exponent)
    side = np.sqrt(30.0 * np.sqrt(d) / 16)
    k[:, :16] = 0.0
    k[block : 2 * block, :16] = side
    q[:, :16] = -side
    q[3::block, :16] = side
    v[block : 2 * block] *= 2.0**octaves
    _check(block, d, heads, bits, q, k, v)


# (the integer kernels carry a factor of 2^26 or 2^13 in the weights up to V scales of 2^40 or 2^90: 46 is on either side of the former)
@pytest.mark.parametrize("block,d,heads", SHAPES)
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("octaves", [-100, -60, 38, 46, 58])
def test_climbing_row_maxima_with_v_of_any_size(block, d, heads, bits, octaves):
    rng = np.random.default_rng(octaves + 200)
    n = BLOCKS * block - 10
    q, k, v = (rng.standard_normal((n, d)) for _ in range(3))
    q, k = 3.0 * np.abs(q), np.abs(k) * np.linspace(0.05, 9.0, n)[:, None]
    _check(block, d, heads, bits, q, k, v * 2.0**octaves)

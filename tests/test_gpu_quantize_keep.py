"""paro_permute_quantize_qkv_keep stores, bit for bit, what the separate reorders and quantizers of Q, K and V store: rows past the
last token included, in every layout of the codes, and values that arithmetic would change (signed zeros, NaN payloads)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bits(t):
    import torch

    return t.view(torch.int16 if t.element_size() == 2 else torch.int32 if t.element_size() == 4 else torch.int8)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,block", [(64, 64), (128, 64), (64, 32), (128, 32)])
@pytest.mark.parametrize("bits", [(8, 8), (8, 4), (4, 4), (4, 8), (16, 16)])
@pytest.mark.parametrize("grid,text", [((3, 5, 7), 0), ((2, 8, 8), 30), ((1, 1, 1), 0)])  # 105 tokens; 128 and 30 text tokens; one
def test_one_launch_equals_the_separate_calls(dtype, d, block, bits, grid, text):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(2, 3, d, *grid, text, block)
    n, npad, k = pb.paro_ntokens(s), pb.paro_npad(s), pb.paro_nblocks(s)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda:0").manual_seed(n + d)
    x = [torch.randn((2, 3, n, d), generator=gen, device="cuda:0").to(tdt) for _ in range(3)]
    x[0][0, 0, 0, :2] = -0.0
    if bits[0] == 16:
        _bits(x[1])[0, 0, 0, 3] = 0x7FA5 if dtype == "bf16" else 0x7F812345  # a NaN with a payload
    ids = np.array([5, 0, 3], np.uint8)

    def outputs():
        ct = [torch.bfloat16 if b == 16 else torch.int8 for b in (bits[0], bits[0], bits[1])]
        lay = (pb.PARO_ROWS, pb.PARO_ROWS, pb.PARO_VT)
        xp = [torch.full((2, 3, npad, d), 7.0, dtype=tdt, device="cuda:0") for _ in range(3)]
        codes = [torch.full(pb.codes_shape(s, b, la), 3, dtype=c, device="cuda:0") for b, la, c in zip((bits[0], bits[0], bits[1]), lay, ct)]
        scales = [torch.full((2, 3, k), 9.0, device="cuda:0") for _ in range(3)]
        return xp, codes, scales

    xp0, c0, s0 = outputs()
    for t in range(3):
        pb.paro_permute(s, ids, x[t], xp0[t])
        pb.paro_quantize(s, bits[t == 2], pb.PARO_VT if t == 2 else pb.PARO_ROWS, xp0[t], c0[t], s0[t])
    xp1, c1, s1 = outputs()
    pb.paro_permute_quantize_qkv_keep(s, *bits, ids, *x, *xp1, c1[0], s1[0], c1[1], s1[1], c1[2], s1[2])
    for a, b in zip(xp0 + c0 + s0, xp1 + c1 + s1):
        assert torch.equal(_bits(a), _bits(b))


@pytest.mark.parametrize("bits", [(8, 8), (4, 4)])
def test_prepare_takes_its_own_reordered_tensors(bits):
    """Without padding an input may be one of the layer's reordered tensors, as long as it is read before it is written."""
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd import workloads as wl
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 2, 64, 2, 8, 8, 0, 64)  # 128 tokens, two blocks
    mask = wl.pack_bitmask(np.ones((2, 2, 2), np.uint8))
    a, b = (ParoAttention(s, [2, 4], mask, *bits, torch.float32) for _ in range(2))
    gen = torch.Generator().manual_seed(1)
    q, k, v = (torch.randn((1, 2, 128, 64), generator=gen).cuda() for _ in range(3))
    want = a.run(q, k, v)
    b.xp[1].copy_(q)
    b.xp[2].copy_(k)
    assert torch.equal(b.run(b.xp[1], b.xp[2], v), want)
    for x, y in zip(a.xp + [a.qc, a.kc, a.vc, a.sq, a.sk, a.sv], b.xp + [b.qc, b.kc, b.vc, b.sq, b.sk, b.sv]):
        assert torch.equal(_bits(x), _bits(y))

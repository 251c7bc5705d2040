"""Integer kernels: Q and K so small that the scale of a block of logits underflows.  Every logit is then 0, attention is the mean of V
over the live keys, and the masked keys of a ragged last block (-inf times that scale) must not turn it into NaN."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2506_16054_amd import workloads as wl
from tests.helpers import check_attention, oracle_head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,d,bits", [(64, 64, (8, 8)), (64, 64, (8, 4)), (64, 64, (4, 8)), (64, 64, (4, 4)), (64, 128, (8, 8)), (64, 128, (8, 4)),
                                          (64, 128, (4, 8)), (32, 64, (8, 8)), (32, 128, (4, 4))])
@pytest.mark.parametrize("gain_q,gain_k", [(2.0**-75, 2.0**-75), (2.0**-75, 2.0**-73), (2.0**-126, 2.0**-100), (2.0**-139, 2.0**-60)])
def test_ragged_block_with_a_vanishing_logit_scale(block, d, bits, gain_q, gain_k):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 1, d, 1, 10, 23, 0, block)  # 230 tokens: the last block has 38 keys of 64, 6 of 32
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    rng = np.random.default_rng(d + block)
    q, k, v = (np.float32(g) * rng.standard_normal((n, d)).astype(np.float32) for g in (gain_q, gain_k, 1.0))
    masks = np.ones((1, kb, kb), bool)
    masks[0, 1, : kb - 1] = False  # a row block with the ragged one alone
    pa = ParoAttention(s, np.zeros(1, np.uint8), wl.pack_bitmask(masks), *bits, torch.float32)
    dev = [torch.from_numpy(x)[None, None].to("cuda:0") for x in (q, k, v)]
    got = pa.run_fused(*dev).clone()
    if bits[0] == 8 and block == 64 and d == 64:  # the same kernel, with Q quantized inside
        assert torch.equal(pa.run_rawq(*dev), got)
    w = SimpleNamespace(F=1, Hg=10, Wg=23, T_text=0, N=n, npad=block * kb, block=block, d=d, bits_qk=bits[0], bits_pv=bits[1])
    ref = oracle_head(w, q, k, v, 0, pa.h_row_ptr[0], pa.h_col_idx, row_blocks=list(range(kb)))
    check_attention(got.cpu().numpy()[0, 0].astype(np.float64), ref["o"], ref["flip_risk"][:n], 2e-2, 1e-2)

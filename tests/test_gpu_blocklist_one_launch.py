"""Bitmask expansion on the device where the one-launch form can go wrong: workgroups that start inside a byte and inside a
head, more row blocks than workgroups, masks that do not start on a 16-byte boundary, bits behind a head's last block,
and either side of the size at which three launches take over."""
import numpy as np
import pytest

from oracle import paro_oracle as po
from tests.test_gpu_prefetch import random_bitmask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nh,k,offset", [(1, 1, 0), (1, 257, 3), (3, 97, 1), (256, 3, 15), (256, 31, 0), (48, 275, 9), (6, 627, 8),
                                         (256, 181, 0), (256, 182, 5), (1, 2896, 2), (1, 2897, 0)])
def test_list_equals_oracle(nh, k, offset):
    import torch

    from paper_2506_16054_amd import binding as pb

    rng = np.random.default_rng([nh, k])
    bits = random_bitmask(rng, nh, k, 0.3, garbage_tail=True)
    ref_ptr, ref_cols = po.mask_to_blocklist(bits, nh, k)
    z = dict(device="cuda:0")
    room = torch.full((bits.size + 64,), 255, dtype=torch.uint8, **z)  # ones in front of and behind the masks
    first = (-room.data_ptr()) % 16 + offset
    d_bits = room[first: first + bits.size].view(bits.shape)
    d_bits.copy_(torch.from_numpy(bits))
    cap = max(1, int(ref_cols.size) - nh)  # the list does not quite fit: its end is dropped, the offsets are whole
    row_ptr = torch.full((nh, k + 1), -7, dtype=torch.int32, **z)
    col_idx = torch.full((cap + 16,), -7, dtype=torch.int32, **z)
    nnz = torch.full((1,), -7, dtype=torch.int32, **z)
    pb.paro_mask_to_blocklist_device(nh, k, d_bits, row_ptr, col_idx[:cap], nnz)
    assert int(nnz.item()) == ref_cols.size
    assert np.array_equal(row_ptr.cpu().numpy(), ref_ptr)
    assert np.array_equal(col_idx.cpu().numpy()[:min(cap, ref_cols.size)], ref_cols[:cap])
    assert bool((col_idx[cap:] == -7).all())

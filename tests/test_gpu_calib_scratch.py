"""Memory of a whole calibration: beyond a stated size the block statistics of one axis order are held at a time, with the
same results."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_large_maps_hold_one_order_at_a_time_and_give_the_same(monkeypatch):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd import pipeline

    s = pb.make_shape(1, 256, 64, 2, 64, 64, 0, 32)  # 256 x 256 blocks per head: the statistics of six orders are 1.2 GB
    n, kb = pb.paro_ntokens(s), pb.paro_nblocks(s)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    q, k = (torch.randn((1, 256, n, 64), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(2))

    def run():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        torch.cuda.reset_peak_memory_stats()
        held = torch.cuda.memory_allocated()
        r = pipeline.calibrate(s, q, k)
        torch.cuda.synchronize()
        return r, torch.cuda.max_memory_allocated() - held

    plane = 4 * 256 * kb * kb
    operands = 2 * 2 * q.numel()
    small, used = run()
    # reordered Q and K, the row statistics, three planes of block statistics; masks, metrics and scales are far below one more
    assert used <= operands + pb.paro_calib_row_stats_bytes(s) + 4 * plane
    monkeypatch.setattr(pipeline, "CALIB_STATS_BYTES", 1 << 40)
    large, used = run()
    assert used >= operands + 18 * plane
    for name in ("perm_ids", "bitmask", "m_sparse", "m_quant", "m_combined", "block_sum"):
        assert torch.equal(small[name], large[name]), name
    assert np.array_equal(small["h_perm_ids"], large["h_perm_ids"])
    assert len(set(small["h_perm_ids"].tolist())) > 1


@pytest.mark.parametrize("B,nh,d,grid,text,block", [(2, 3, 64, (3, 7, 9), 0, 32), (1, 2, 128, (1, 16, 16), 64, 64), (3, 1, 64, (1, 5, 9), 0, 64)])
def test_one_order_at_a_time_gives_the_same(monkeypatch, B, nh, d, grid, text, block):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd import pipeline

    s = pb.make_shape(B, nh, d, *grid, text, block)
    gen = torch.Generator(device="cuda:0").manual_seed(d + block)
    q, k = (torch.randn((B, nh, pb.paro_ntokens(s), d), generator=gen, device="cuda:0") for _ in range(2))
    want = pipeline.calibrate(s, q, k, density=0.4)
    monkeypatch.setattr(pipeline, "CALIB_STATS_BYTES", 0)
    got = pipeline.calibrate(s, q, k, density=0.4)
    for name in ("perm_ids", "bitmask", "m_sparse", "m_quant", "m_combined", "block_sum"):
        assert torch.equal(got[name], want[name]), name

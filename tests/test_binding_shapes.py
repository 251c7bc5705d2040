"""The binding keeps what follows from a shape by the shape's numbers: a refusal is not kept, a changed shape is another.
Its stream handle does not hang on a function that torch does not promise."""
import types

import pytest

from paper_2506_16054_amd import binding as pb


@pytest.mark.parametrize("block", [32, 64])
def test_a_shape_that_changes_gets_its_own_counts(block):
    s = pb.make_shape(1, 2, 64, 3, 5, 7, 0, block)  # 105 tokens
    k = -(-105 // block)
    assert (pb.paro_ntokens(s), pb.paro_nblocks(s), pb.paro_npad(s)) == (105, k, k * block)
    assert pb.codes_shape(s, 4, pb.PARO_ROWS) == (1, 2, k * block, 32) and pb.codes_shape(s, 4, pb.PARO_VT) == (1, 2, k, 64, block // 2)
    s.F = 6
    assert pb.paro_ntokens(s) == 210 and pb.codes_shape(s, 8, pb.PARO_VT) == (1, 2, -(-210 // block), 64, block)


def test_a_refused_shape_is_refused_every_time():
    bad = pb.make_shape(1, 2, 64, 3, 5, 7, 0, 48)
    for _ in range(2):
        for f in (pb.paro_ntokens, pb.paro_nblocks, pb.paro_npad):
            with pytest.raises(pb.ParoError) as e:
                f(bad)
            assert e.value.status == pb.PARO_EUNSUPPORTED  # blocks of 48 are not built
    bad.block = 64
    assert pb.paro_ntokens(bad) == 105


def test_stream_without_the_private_function(monkeypatch):
    import torch

    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4711))
    assert pb._stream() == 4711

"""The per-layer calls made by the native module: the same bytes as through the binding's own checks, and the module declines
(the binding then raises, or accepts) whatever is not a plain contiguous tensor of the expected shape and type."""
import types

import numpy as np
import pytest
import torch

from paper_2506_16054_amd import binding as pb
from paper_2506_16054_amd import workloads as wl
from paper_2506_16054_amd.pipeline import ParoAttention

class Sub(torch.Tensor):
    pass


NONE = types.SimpleNamespace(**{name: (lambda *a: None) for name in pb.FASTCALL})


def _layer(bits_qk, bits_pv, dtype, block=64, d=64, device="cuda:0"):
    s = pb.make_shape(1, 2, d, 3, 5, 7, 11, block)
    k = pb.paro_nblocks(s)
    live = np.random.default_rng(3).random((2, k, k)) < 0.6
    live[:, np.arange(k), np.arange(k)] = True
    bits = wl.pack_bitmask(live.astype(np.uint8))
    pa = ParoAttention(s, [1, 4], bits, bits_qk, bits_pv, dtype, device)
    g = torch.Generator().manual_seed(5)
    x = [torch.randn((1, 2, pa.N, d), generator=g).to(device, dtype) for _ in range(3)]
    return pa, bits, x


@pytest.mark.parametrize("name", pb.FASTCALL)
def test_module_declines_host_arguments(name):
    """Nothing but the right objects is taken: host tensors, numbers, None and a wrong count go on to the binding's checks."""
    f = getattr(pb._native(), name)
    s = pb.make_shape(1, 2, 64, 3, 5, 7, 11, 64)
    for a in (torch.zeros(4), None, 3, "x", np.zeros(2, np.uint8)):
        for n in (4, 6, 13, 14, 16):
            assert f(*([s, 8, 8] + [a] * n)[:n]) is None
    assert f() is None


def test_module_is_missing(monkeypatch, tmp_path):
    monkeypatch.setattr(pb, "_fast", None)
    monkeypatch.setattr(pb, "lib", lambda: None)
    monkeypatch.setattr(pb, "__file__", str(tmp_path / "binding.py"))
    with pytest.raises(pb.ParoError, match="paro_fastcall.so is missing"):
        pb._native()


def _calls_without_module(monkeypatch, match):
    """The per-layer calls reach the binding's own checks (which refuse these arguments) after one warning."""
    monkeypatch.setattr(pb, "_fast", None)
    s = pb.make_shape(1, 2, 64, 3, 5, 7, 11, 64)
    with pytest.warns(RuntimeWarning, match=match):
        with pytest.raises(pb.ParoError, match="must be"):
            pb.paro_unpermute(s, [0, 0], torch.zeros(4), torch.zeros(4))
    for name in pb.FASTCALL:
        assert getattr(pb._fast, name)(1, 2, 3) is None


def test_calls_go_on_without_the_module(monkeypatch, tmp_path):
    pb.lib()
    monkeypatch.setattr(pb, "__file__", str(tmp_path / "binding.py"))
    _calls_without_module(monkeypatch, "paro_fastcall.so is missing")


def test_module_for_another_torch_is_not_used(monkeypatch):
    pb._native()
    monkeypatch.setattr(torch, "__version__", "0.0.0")
    _calls_without_module(monkeypatch, "not 0.0.0")


def test_build_goes_on_without_a_compiler(monkeypatch, tmp_path, capfd):
    from paper_2506_16054_amd import build

    stale = tmp_path / build.FASTCALL_LIBNAME
    for cxx in ("no-such-compiler", "false"):
        monkeypatch.setenv("CXX", cxx)
        stale.write_bytes(b"of an earlier build")
        assert build.build_fastcall(str(tmp_path)) is None
        assert not stale.exists() and "native module" in capfd.readouterr().err


@pytest.mark.gpu
@pytest.mark.parametrize("bits_qk,bits_pv", pb.QKV_BITS)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_same_bytes_as_the_binding(monkeypatch, bits_qk, bits_pv, dtype):
    pa, bits, x = _layer(bits_qk, bits_pv, dtype)
    row_ptr, cols = torch.empty_like(pa.row_ptr), torch.empty_like(pa.col_idx)

    def spoil():
        """Nothing that a call is to write holds what an earlier one wrote there."""
        for t in (row_ptr, cols, pa.op, pa.o, *pa.xp, pa.qc, pa.kc, pa.vc, pa.sq, pa.sk, pa.sv, *pa._fused_buffers()):
            t.fill_(3)

    def once():
        spoil()
        pb.paro_mask_to_blocklist_device(2, pa.k, torch.from_numpy(bits).to("cuda:0"), row_ptr, cols)
        pa.use_blocklist(row_ptr, cols, pa.row_order)
        out = [row_ptr.clone(), cols.clone(), pa.run(*x).clone(), pa.op.clone()]
        out += [t.clone() for t in (*pa.xp, pa.qc, pa.kc, pa.vc, pa.sq, pa.sk, pa.sv)]
        spoil()
        row_ptr.copy_(out[0]), cols.copy_(out[1])
        pa.prepare_fused_qkv(*x)
        out += [t.clone() for t in (*pa._fused_buffers(), pa.vc, pa.sq, pa.sk, pa.sv)]
        return out + [pa.attend_fused().clone()]

    pa.row_order = torch.from_numpy(pa.h_row_order).to("cuda:0")
    calls = []
    native = pb._native()

    def watched(name):
        def call(*a):
            calls.append((name, getattr(native, name)(*a)))
            return calls[-1][1]
        return call

    monkeypatch.setattr(pb, "_fast", types.SimpleNamespace(**{name: watched(name) for name in pb.FASTCALL}))
    got = once()
    assert calls and all(status == pb.PARO_OK for _, status in calls)
    monkeypatch.setattr(pb, "_fast", NONE)
    for a, b in zip(got, once(), strict=True):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
def test_declined_and_refused_on_the_device():
    pa, bits, x = _layer(8, 8, torch.float32)
    f = pb._native().paro_unpermute
    op, o = pa.op, pa.o
    assert f(pa.s, pa.perm_ids, op, o) == pb.PARO_OK
    wide = torch.empty((1, 2, pa.npad, 128), device="cuda:0")[..., :64]
    for a, b, ids in ((wide, o, pa.perm_ids), (op[:, :, 1:], o, pa.perm_ids), (op.bfloat16(), o, pa.perm_ids), (op.half(), o.half(), pa.perm_ids),
                      (op, o, pa.perm_ids.astype(np.int64)), (op, o, pa.perm_ids[:1]), (op, o, bytes(pa.perm_ids)), (op, o, [1, 4]),
                      (op, o, np.array([1, 9, 4], np.uint8)[::2]), (op.as_subclass(Sub), o, pa.perm_ids), (op.cpu(), o, pa.perm_ids)):
        assert f(pa.s, ids, a, b) is None
    # what the module takes, the library still checks; what it leaves, the binding accepts or refuses as before
    for ids in ([1, 9], np.array([1, 9], np.uint8)):
        with pytest.raises(pb.ParoError):
            pb.paro_unpermute(pa.s, ids, op, o)
    with pytest.raises(pb.ParoError):
        pb.paro_unpermute(pa.s, pa.perm_ids, wide, o)
    pb.paro_unpermute(pa.s, [1, 4], op.as_subclass(Sub), o)
    seen = []
    torch.func.vmap(lambda t: seen.append(f(pa.s, pa.perm_ids, t, o)) or t)(op[None])
    assert seen == [None]


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_calls_follow_the_current_stream(monkeypatch, native):
    """Inputs that arrive late on a side stream: a call on any other stream would read what was there before."""
    pa, bits, x = _layer(8, 8, torch.float32)
    want_steps = pa.run(*x).clone()
    pa.prepare_fused_qkv(*x)
    want_fused = pa.attend_fused().clone()
    late = [torch.zeros_like(t) for t in x]
    monkeypatch.setattr(pb, "_fast", pb._native() if native else NONE)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for want, call in ((want_steps, lambda: pa.run(*late)), (want_fused, lambda: (pa.prepare_fused_qkv(*late), pa.attend_fused())[1])):
            [t.zero_() for t in late]
            torch.cuda._sleep(20_000_000)  # some 10 ms
            [t.copy_(s) for t, s in zip(late, x)]
            o = call().clone()
            side.synchronize()
            assert torch.equal(o, want)


@pytest.mark.gpu
def test_two_threads_with_a_layer_and_a_stream_each():
    import threading

    layers = [_layer(8, 8, torch.float32), _layer(4, 4, torch.bfloat16)]
    want = [(pa.run(*x).clone(), (pa.prepare_fused_qkv(*x), pa.attend_fused())[1].clone()) for pa, _, x in layers]
    torch.cuda.synchronize()
    wrong, start = [], threading.Barrier(2)

    def work(i):
        pa, _, x = layers[i]
        start.wait()
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(50):
                steps = pa.run(*x).clone()
                pa.prepare_fused_qkv(*x)
                fused = pa.attend_fused().clone()
                torch.cuda.current_stream().synchronize()
                if not (torch.equal(steps, want[i][0]) and torch.equal(fused, want[i][1])):
                    wrong.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert wrong == []

"""The calls that put several quantizers into one grid: K and V alone, and Q, K, V with the channel mean of K removed.  Mean,
codes and scales are those of the separate calls bit for bit, through the native module and through ctypes, nothing beside the
outputs is written, and what the separate calls refuse is refused."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BITS = [(8, 8), (8, 4), (4, 4), (4, 8)]


@pytest.fixture(params=["native", "ctypes"])
def route(request, monkeypatch):
    from paper_2506_16054_amd import binding as pb

    monkeypatch.setattr(pb, "_fast", pb._native() if request.param == "native" else pb._NoNative)
    return request.param


def _buffers(pb, s, bits_qk, bits_pv, fill):
    import torch

    k = pb.paro_nblocks(s)
    codes = [torch.full(pb.codes_shape(s, b, lay), fill, dtype=torch.int8, device="cuda:0")
             for b, lay in ((bits_qk, pb.PARO_ROWS), (bits_qk, pb.PARO_ROWS), (bits_pv, pb.PARO_VT))]
    scales = [torch.full((s.B, s.nh, k), float(fill), device="cuda:0") for _ in range(3)]
    return codes, scales


@pytest.mark.parametrize("block,d", [(64, 64), (64, 128), (32, 64), (32, 128)])
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_same_bits_as_the_separate_calls(route, block, d, bits, dtype):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(2, 3, d, 3, 7, 11, 0, block)  # 231 tokens, ragged in both block sizes
    gen = torch.Generator(device="cuda:0").manual_seed(block + d + sum(bits))
    q, k, v = (torch.randn((2, 3, 231, d), generator=gen, device="cuda:0").to(getattr(torch, dtype)) for _ in range(3))
    k += torch.arange(d, device="cuda:0").to(k.dtype) / 16
    ids = np.array([0, 3, 5], np.uint8)
    qk, pv = bits
    want, ws = _buffers(pb, s, qk, pv, 1)
    mean = torch.zeros((2, 3, d), device="cuda:0")
    pb.paro_k_channel_mean(s, k, mean)
    pb.paro_permute_quantize(s, qk, pb.PARO_ROWS, ids, q, want[0], ws[0])
    pb.paro_permute_quantize(s, pv, pb.PARO_VT, ids, v, want[2], ws[2])
    for smoothed in (True, False):
        if smoothed:
            pb.paro_permute_quantize_smoothed(s, qk, ids, k, mean, want[1], ws[1])
        else:
            pb.paro_permute_quantize(s, qk, pb.PARO_ROWS, ids, k, want[1], ws[1])
        got, gs = _buffers(pb, s, qk, pv, 2)
        got_mean = torch.full_like(mean, 7.0)
        if smoothed:
            pb.paro_permute_quantize_qkv_smoothed(s, qk, pv, ids, q, k, v, got_mean, got[0], gs[0], got[1], gs[1], got[2], gs[2])
            assert torch.equal(got_mean, mean)
        else:
            pb.paro_permute_quantize_kv(s, qk, pv, ids, k, v, got[1], gs[1], got[2], gs[2])
            assert bool((got[0] == 2).all()) and bool((gs[0] == 2).all())
        for i in range(0 if smoothed else 1, 3):
            assert torch.equal(got[i], want[i]) and torch.equal(gs[i], ws[i]), (smoothed, i)


def test_whole_forms_on_both_routes(route):
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd import workloads as wl
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 2, 64, 2, 10, 12, 0, 64)
    pa = ParoAttention(s, np.array([1, 4], np.uint8), wl.pack_bitmask(np.ones((2, 4, 4), bool)), 8, 4, torch.float32)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    q, k, v = (torch.randn((1, 2, 240, 64), generator=gen, device="cuda:0") for _ in range(3))
    fused = pa.run_fused(q, k, v).clone()
    assert torch.equal(pa.run_rawq(q, k, v), fused)
    # tensors of different types go through the separate calls, as they did
    mixed = pa.run_rawq(q, k, v.to(torch.bfloat16)).clone()
    assert torch.equal(pa.run_fused(q, k, v.to(torch.bfloat16).float()), mixed)
    smooth = pa.run_fused_smooth_k(q, k, v).clone()
    mixed = pa.run_fused_smooth_k(q.to(torch.bfloat16), k, v).clone()
    assert torch.equal(pa.run_fused_smooth_k(q.to(torch.bfloat16).float(), k, v), mixed)
    fq, fk = pa._fused_buffers()
    pb.paro_k_channel_mean(s, k, pa.k_mean)
    pb.paro_permute_quantize(s, 8, pb.PARO_ROWS, pa.perm_ids, q, fq, pa.sq)
    pb.paro_permute_quantize_smoothed(s, 8, pa.perm_ids, k, pa.k_mean, fk, pa.sk)
    pb.paro_permute_quantize(s, 4, pb.PARO_VT, pa.perm_ids, v, pa.vc, pa.sv)
    assert torch.equal(pa.attend_fused(), smooth)


def test_refusals(route):
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(1, 1, 64, 1, 8, 8, 0, 64)
    x = torch.zeros((1, 1, 64, 64), device="cuda:0")
    codes, scales = _buffers(pb, s, 8, 8, 0)
    mean = torch.zeros((1, 1, 64), device="cuda:0")
    ids = np.zeros(1, np.uint8)
    full = lambda c=codes, sc=scales, m=mean, b=(8, 8), p=ids, t=x: pb.paro_permute_quantize_qkv_smoothed(s, *b, p, t, t, t, m, c[0], sc[0], c[1], sc[1], c[2], sc[2])
    full()
    for bad in (lambda: full(c=[codes[0], codes[0], codes[2]]), lambda: full(b=(8, 16)), lambda: full(p=np.full(1, 6, np.uint8)), lambda: full(m=mean[:, :, :32]),
                lambda: full(t=x[:, :, :32]), lambda: full(t=x.double()),
                lambda: pb.paro_permute_quantize_kv(s, 8, 8, ids, x, x.to(torch.bfloat16), codes[1], scales[1], codes[2], scales[2]),
                lambda: pb.paro_permute_quantize_kv(s, 8, 8, ids, x, x, codes[1], scales[1], codes[1].view(1, 1, 1, 64, 64), scales[2])):
        with pytest.raises(pb.ParoError):
            bad()


@pytest.mark.parametrize("heads,d,grid,bits_qk,dtype", [
    (3, 64, (1, 63, 65), 4, "bfloat16"),     # 4095 tokens: the mean by channels
    (3, 64, (1, 64, 64), 4, "bfloat16"),     # 4096: by sums, 8 spans of 512
    (3, 128, (1, 17, 241), 4, "bfloat16"),   # 4097: a span of one token
    (100, 64, (1, 64, 65), 8, "bfloat16"),   # as many spans as 512 workgroups allow
    (2, 128, (13, 30, 45), 8, "bfloat16"),
    (3, 64, (1, 23, 89), 4, "float32"),      # 2047
    (3, 64, (1, 32, 64), 4, "float32"),      # 2048
    (3, 128, (1, 3, 683), 4, "float32"),     # 2049
    (260, 64, (1, 32, 65), 4, "float32"),    # one span per head
])
def test_mean_by_sums_is_the_mean(heads, d, grid, bits_qk, dtype):
    """Where the rows are long the mean's partial sums meet in the buffer of Q's codes: mean, codes and scales as by the separate calls."""
    import torch

    from paper_2506_16054_amd import binding as pb

    s = pb.make_shape(2, heads // 2, d, *grid, 0, 32) if heads > 256 else pb.make_shape(1, heads, d, *grid, 0, 32)
    n = grid[0] * grid[1] * grid[2]
    gen = torch.Generator(device="cuda:0").manual_seed(n + d)
    q, v = (torch.randn((s.B, s.nh, n, d), generator=gen, device="cuda:0").to(getattr(torch, dtype)) for _ in range(2))
    k = (torch.randn((s.B, s.nh, n, d), generator=gen, device="cuda:0") + 4 * torch.randn((s.B, s.nh, 1, d), generator=gen, device="cuda:0")).to(q.dtype)
    perm = (np.arange(s.nh) % 6).astype(np.uint8)
    codes, scales = _buffers(pb, s, bits_qk, 8, 5)
    mean = torch.full((s.B, s.nh, d), 7.0, device="cuda:0")
    pb.paro_permute_quantize_qkv_smoothed(s, bits_qk, 8, perm, q, k, v, mean, codes[0], scales[0], codes[1], scales[1], codes[2], scales[2])
    want_codes, want_scales = _buffers(pb, s, bits_qk, 8, 6)
    want_mean = torch.empty_like(mean)
    pb.paro_k_channel_mean(s, k, want_mean)
    pb.paro_permute_quantize(s, bits_qk, pb.PARO_ROWS, perm, q, want_codes[0], want_scales[0])
    pb.paro_permute_quantize_smoothed(s, bits_qk, perm, k, want_mean, want_codes[1], want_scales[1])
    pb.paro_permute_quantize(s, 8, pb.PARO_VT, perm, v, want_codes[2], want_scales[2])
    assert torch.equal(mean, want_mean)
    assert torch.equal(mean, k.double().mean(dim=2).to(torch.float32).to(torch.bfloat16).float())
    for a, b in zip(codes + scales, want_codes + want_scales):
        assert torch.equal(a, b)


def _long_layer(bits, seed):
    """2048 fp32 tokens: the channel mean is made of partial sums that meet in Q's codes."""
    import torch

    from paper_2506_16054_amd import binding as pb
    from paper_2506_16054_amd import workloads as wl
    from paper_2506_16054_amd.pipeline import ParoAttention

    s = pb.make_shape(1, 3, 64, 1, 32, 64, 0, 64)
    live = np.random.default_rng(seed).random((3, 32, 32)) < 0.4
    live[:, np.arange(32), np.arange(32)] = True
    pa = ParoAttention(s, np.array([0, 2, 5], np.uint8), wl.pack_bitmask(live), *bits, torch.float32)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    x = [torch.randn((1, 3, 2048, 64), generator=gen, device="cuda:0") for _ in range(3)]
    x[1] += 3.0 * torch.randn((1, 3, 1, 64), generator=gen, device="cuda:0")
    return pa, x


def _forms(pa):
    return [pa.run_fused_smooth_k] + ([pa.run_rawq] if pa.can_fuse_q else [])


@pytest.mark.parametrize("bits", [(8, 8), (4, 8)])
def test_inputs_that_arrive_late_on_a_side_stream(route, bits, monkeypatch):
    """A call on any other stream, or sums read from another stream's scratch, would see what was there before."""
    import types

    import torch

    from paper_2506_16054_amd import binding as pb

    pa, x = _long_layer(bits, 1)
    want = [form(*x).clone() for form in _forms(pa)]
    taken = []
    if route == "native":  # the module takes these calls as they stand
        native = pb._native()
        watched = {name: (lambda f: lambda *a: taken.append(f(*a)) or taken[-1])(getattr(native, name)) for name in pb.FASTCALL}
        monkeypatch.setattr(pb, "_fast", types.SimpleNamespace(**watched))
    late = [torch.zeros_like(t) for t in x]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for form, o in zip(_forms(pa), want):
            [t.zero_() for t in late]
            [t.fill_(7) for t in (*pa._fused_buffers(), pa.vc, pa.sq, pa.sk, pa.sv, pa.k_mean)]
            torch.cuda._sleep(20_000_000)  # some 10 ms
            [t.copy_(s) for t, s in zip(late, x)]
            got = form(*late).clone()
            side.synchronize()
            assert torch.equal(got, o)
    assert route != "native" or (len(taken) == 2 * len(want) and all(status == pb.PARO_OK for status in taken))


def test_two_threads_with_a_layer_and_a_stream_each(route):
    import threading

    import torch

    layers = [_long_layer((8, 8), 2), _long_layer((4, 4), 3)]
    want = [[form(*x).clone() for form in _forms(pa)] for pa, x in layers]
    torch.cuda.synchronize()
    wrong, start = [], threading.Barrier(2)

    def work(i):
        pa, x = layers[i]
        start.wait()
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(50):
                got = [form(*x).clone() for form in _forms(pa)]
                torch.cuda.current_stream().synchronize()
                if not all(torch.equal(a, b) for a, b in zip(got, want[i])):
                    wrong.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert wrong == []

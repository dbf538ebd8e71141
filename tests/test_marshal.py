"""The binding's extension module: what it does not take it leaves to the
Python function (CPU), and the calls it makes give the ctypes path's bits and
errors for every optional argument, other streams and refused arguments (GPU)."""
import os

import pytest

import paper_2304_11267_amd as sd
from paper_2304_11267_amd import binding


@pytest.fixture(scope="module")
def native():
    if not os.path.exists(binding.library_path()):
        pytest.skip("library not built")
    sd.load_library()
    assert binding._native is not None, "the extension module is not built"
    return binding._native


def test_cpu_tensors_and_odd_arguments_are_left_to_python(native):
    import torch
    t = torch.zeros(1, 1, 8, 32, dtype=torch.float16)
    fn = binding._fn["sdattn_forward"]
    assert native.forward(fn, t, t, t, t, 0.1, None) is None
    assert native.forward(fn, t, t, t, t) is None
    assert native.forward(fn, None, 3, "x", t, 0.1, None) is None
    assert native.forward() is None
    for name in ("forward_ex", "softmax_rows", "logits", "softmax_pv", "attention_block", "attention_block_kv",
                 "group_norm", "geglu", "conv3x3"):
        assert getattr(native, name)(fn, t, t, t, t, t, t, t, t, t, 1, 0.1, None) is None
    with pytest.raises(ValueError, match="GPU tensor"):
        sd.forward(t, t, t, torch.empty_like(t), 0.1)


@pytest.mark.gpu
def test_same_bits_and_errors_as_ctypes(native, monkeypatch):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(3)

    def rnd(*shape, dt=torch.float16):
        return torch.randn(*shape, device="cuda", generator=g).to(dt)

    q, k, v = rnd(2, 8, 70, 40), rnd(2, 8, 90, 40), rnd(2, 8, 90, 40)
    x, ctx, wq, wk, wv, wo, bo = (rnd(2, 70, 320), rnd(2, 77, 768), rnd(320, 320), rnd(320, 768), rnd(320, 768),
                                  rnd(320, 320), rnd(320))
    kh, vh = rnd(2, 8, 77, 40), rnd(2, 8, 77, 40)
    u, img = rnd(36, 16, 24), rnd(2, 24, 9, 12)
    side = torch.cuda.Stream()

    def calls(stream):
        on = stream or torch.cuda.current_stream()
        on.wait_stream(torch.cuda.current_stream())

        def now(t):   # t's values after the calls so far
            on.synchronize()
            return t.clone()

        o = torch.full_like(q, 7.0)
        ls = torch.empty(2, 8, 70, 2, device="cuda")
        a = torch.empty(2, 8, 70, 90, dtype=torch.float32, device="cuda")
        p = torch.empty(2 * 8 * 70, 90, device="cuda")
        y, y2 = torch.empty_like(x), torch.empty_like(x)
        ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
        c = torch.empty(2, 16, 9, 12, dtype=torch.float16, device="cuda")
        n, n2 = torch.empty_like(img), torch.empty_like(img)
        e = torch.empty(2, 70, 160, dtype=torch.float16, device="cuda")
        torch.cuda.synchronize()
        out = [now(sd.forward(q, k, v, o, 0.2, stream))]
        o.fill_(7.0)
        torch.cuda.synchronize()
        out += [now(sd.forward_ex(q, k, v, o, 0.2, ls=ls, stream=stream)), now(ls)]
        out += [sd.logits(q, k, a, 0.2, stream)]
        out += [now(sd.softmax_rows(a.view(-1, 90), ls.view(-1, 2), p, 1.0, stream)), p]
        out += [sd.softmax_pv(a, ls, v, torch.empty_like(q), stream)]
        out += [sd.attention_block(x, ctx, wq, wk, wv, wo, bo, y, ws, 8, 0.1, stream)]
        out += [sd.attention_block_kv(x, wq, kh, vh, wo, None, y2, ws, 0.1, stream)]
        out += [sd.group_norm(img, 8, n, stream=stream), sd.group_norm(img, 8, n2, rnd_c, None, 1e-3, stream)]
        out += [sd.geglu(x, e, stream), sd.conv3x3(img, u, c, ws, stream=stream)]
        torch.cuda.synchronize()
        return out

    def reads_in_order(call, src):
        """Whether call(stream), on a side stream, sees the values that a copy queued there
        before it gives src."""
        old, new = src.clone(), src.flip(0).contiguous()
        want = call(None, new).clone()
        for stream, current in ((side, torch.cuda.current_stream()), (None, side)):
            src.copy_(old)
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                torch.cuda._sleep(10_000_000)   # some milliseconds
                src.copy_(new)
            with torch.cuda.stream(current):
                got = call(stream, src)
            torch.cuda.synchronize()
            if not torch.equal(got, want):
                return False
        src.copy_(old)
        torch.cuda.synchronize()
        return True

    rnd_c = rnd(24)
    torch.cuda.synchronize()
    outs = [torch.empty_like(t) for t in (q, x, img)]
    big = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    assert reads_in_order(lambda s, t: sd.forward(t, k, v, outs[0], 0.2, s), q)
    assert reads_in_order(lambda s, t: sd.forward_ex(t, k, v, outs[0], 0.2, stream=s), q)
    assert reads_in_order(lambda s, t: sd.attention_block(t, ctx, wq, wk, wv, wo, bo, outs[1], big, 8, 0.1, s), x)
    assert reads_in_order(lambda s, t: sd.group_norm(t, 8, outs[2], stream=s), img)
    fast = [calls(None), calls(side)]
    with torch.cuda.stream(side):
        fast.append(calls(None))
    monkeypatch.setattr(binding, "_native", None)
    slow = calls(None)
    for got in fast:
        assert len(got) == len(slow) and all(torch.equal(a, b) for a, b in zip(got, slow))
    # a size that the library refuses, and shapes that the binding refuses
    bad = rnd(1, 1, 8, 12)
    for mod in (native, None):
        monkeypatch.setattr(binding, "_native", mod)
        with pytest.raises(sd.SdattnError) as err:
            sd.forward(bad, bad, bad, torch.empty_like(bad), 0.1)
        assert err.value.status == sd.STATUS_UNSUPPORTED
        with pytest.raises(ValueError, match="v has shape"):
            sd.forward(q, k, v[:, :, :80].contiguous(), torch.empty_like(q), 0.1)
        with pytest.raises(ValueError, match="contiguous"):
            sd.forward(q.transpose(2, 3).contiguous().transpose(2, 3), k, v, torch.empty_like(q), 0.1)
        with pytest.raises(TypeError, match="k is"):
            sd.forward(q, k.bfloat16(), v, torch.empty_like(q), 0.1)

"""The native marshalling of the binding against the ctypes path.

The same calls are made through the native functions and with the ctypes path
alone.  Both must pass the same arguments on, so every output is bit-identical;
a failed check or a return code of the library raises the same error on both.
What the native functions return says which path served a call: the library's
code, or None where they hand it on (lengths and positions in numpy arrays).
"""
import contextlib
import ctypes
import weakref

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _calls(mad, as_seq):
    """name -> (output tensors, call) over the entry points with both paths; `as_seq` makes the host sequences."""
    from paper_2608_30252_amd import synth
    dev = "cuda"
    n = lambda shape, seed, std=1.0, dt=torch.bfloat16: synth.normal(shape, seed, std=std, dtype=dt).to(dev)
    B, Hq, Hkv, d, D, T = 3, 8, 2, 64, 2048, 3
    q, mk, mv = n((B, Hq, d), 1), n((B, Hkv, 40, d), 2), n((B, Hkv, 40, d), 3)
    wk, wv, kn, vn = n((B, Hkv, 50, d), 4), n((B, Hkv, 50, d), 5), n((B, Hkv, d), 6), n((B, Hkv, d), 7)
    mem, win = mad.KV(mk, mv, as_seq([7, 0, 31])), mad.KV(wk, wv, as_seq([20, 49, 3]), as_seq([45, 1, 9]))
    o, l = torch.empty_like(q), torch.empty(B, Hq, device=dev)
    yield "decode", [o, l, wk, wv], lambda: mad.draft_decode_attn(q, mem, win, kn, vn, o, l)
    o2, l2 = torch.empty_like(q), torch.empty(B, Hq, device=dev)
    yield "step", [o2, l2, wk, wv], lambda: mad.draft_step_attn(q, mem, win, kn, vn, as_seq([1, 2, 0]), o2, l2, 0.2)
    x, w = n((B, 2, D), 8), n((2 * Hkv * d, D), 9, 0.02)
    yield "update", [mk, mv], lambda: mad.memory_update(x, w, [as_seq([3 * b, 9]) for b in range(B)],
                                                        mad.KV(mk, mv, as_seq([7, 0, 31])), fire=as_seq([1, 0, 1]))
    qv, vk, vv = n((B, T, Hq, d), 10), n((B, Hkv, 64, d), 11), n((B, Hkv, 64, d), 12)
    ov, lv = torch.empty_like(qv), torch.empty(B, T, Hq, device=dev)
    yield "verify", [ov, lv], lambda: mad.verify_attn(qv, mad.KV(vk, vv, as_seq([3, 64, 40])), ov, lv)
    vt = vv.transpose(2, 3).contiguous()
    ot, lt = torch.empty_like(qv), torch.empty(B, T, Hq, device=dev)
    yield "verify_vt", [ot, lt], lambda: mad.verify_attn_vt(qv, vk, vt, as_seq([3, 64, 40]), ot, lt)
    xr, gm, wq = n((2, D), 13), n((D,), 14), n(((Hq + 2 * Hkv) * d, D), 15, 0.02)
    qo, ko, vo, xn = (torch.empty(s, dtype=torch.bfloat16, device=dev) for s in ((2, Hq, d), (2, Hkv, d), (2, Hkv, d), (2, D)))
    yield "qkv", [qo, ko, vo, xn], lambda: mad.rmsnorm_qkv_rope(xr, gm, wq, as_seq([5, 70]), Hq, Hkv, d, qo, ko, vo, xn)
    # (no host sequence in these)
    wo, res, lo = n((256, D), 16, 0.02), n((2, 256), 17), torch.empty(2, 256, dtype=torch.bfloat16, device=dev)
    yield "linear", [lo], lambda: mad.linear_residual(xr, wo, res, lo)
    wg, so = n((2 * 4096, D), 18, 0.02), torch.empty(2, 4096, dtype=torch.bfloat16, device=dev)
    yield "swiglu", [so], lambda: mad.rmsnorm_swiglu(xr, gm, wg, so)
    V = 5000
    for rows in (1, 4):
        draft = torch.randint(0, V, (B, rows - 1), dtype=torch.int32, device=dev, generator=torch.Generator(dev).manual_seed(19)) if rows > 1 else None
        for dt in (torch.float32, torch.bfloat16):
            lg, na, nt = n((B, rows, V), 20, dt=dt), *(torch.empty(B, dtype=torch.int32, device=dev) for _ in range(2))
            yield "greedy", [na, nt], lambda: mad.accept_greedy(lg, draft, na, nt)
    pp, pq = (torch.softmax(n((B, r, V), 21 + r, dt=torch.float32), -1) for r in (4, 3))
    u = torch.rand(B, 4, device=dev, generator=torch.Generator(dev).manual_seed(22))
    sa, st = (torch.empty(B, dtype=torch.int32, device=dev) for _ in range(2))
    yield "stoch", [sa, st], lambda: mad.accept_stochastic(pp, pq, draft, u, sa, st)


class _Recorded:
    """The native module, and what its functions returned."""

    def __init__(self, fast):
        self.fast, self.returned = fast, []

    def __getattr__(self, name):
        def call(*args):
            self.returned.append((name, getattr(self.fast, name)(*args)))
            return self.returned[-1][1]
        return call


def test_native_and_ctypes_marshalling_agree(monkeypatch):
    import paper_2608_30252_amd as mad
    native, ctypes_only = _Recorded(mad._fast()), mad._CtypesOnly()
    served = set()
    for (name, a, f), (_, b, g), (_, _, h) in zip(_calls(mad, list), _calls(mad, list), _calls(mad, np.array)):
        for call, fast in ((f, native), (g, ctypes_only), (f, native), (g, ctypes_only)):
            monkeypatch.setattr(mad, "_FAST", fast)   # the first native call may find no workspace yet
            call()
        torch.cuda.synchronize()
        function, rc = native.returned[-1]
        assert rc == mad.MAD_OK, f"{name}: {function} returned {rc}"   # served natively, not handed on (None)
        served.add(function)
        for i, (s, t) in enumerate(zip(a, b)):
            bits = torch.int16 if s.dtype == torch.bfloat16 else torch.int32
            assert torch.equal(s.view(bits), t.view(bits)), f"{name}: output {i}"
        if name in ("decode", "step", "update", "verify", "verify_vt", "qkv"):   # lengths in arrays are handed on
            monkeypatch.setattr(mad, "_FAST", native)
            h()
            assert native.returned[-1] == (function, None), name
    assert served == {"attn", "update", "verify", "verify_vt", "greedy", "stoch", "qkv", "linear", "swiglu"}


def test_a_side_stream_has_its_own_workspace(monkeypatch):
    import paper_2608_30252_amd as mad
    native = _Recorded(mad._fast())
    name, (out, lse, *_), f = next(_calls(mad, list))
    f()
    torch.cuda.synchronize()
    want = out.clone(), lse.clone()
    out.zero_()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        f()   # allocates the stream's workspace through the ctypes path
        monkeypatch.setattr(mad, "_FAST", native)
        f()
        side.synchronize()
        keys = [k for k in mad._default_ws if k[1] == side.cuda_stream]
    assert native.returned == [("attn", mad.MAD_OK)] and len(keys) == 1
    assert torch.equal(out.view(torch.int16), want[0].view(torch.int16)) and torch.equal(lse, want[1])


@pytest.mark.parametrize("as_seq", [list, np.array])
def test_errors_are_the_same_on_both_paths(as_seq):
    import paper_2608_30252_amd as mad
    q = torch.zeros(2, 8, 64, dtype=torch.bfloat16, device="cuda")
    k = torch.zeros(2, 2, 16, 64, dtype=torch.bfloat16, device="cuda")
    o, l = torch.empty_like(q), torch.empty(2, 8, device="cuda")
    with pytest.raises(mad.MadError, match="exceeds cap") as e:
        mad.draft_decode_attn(q, mad.KV(k, k, as_seq([17, 1])), None, None, None, o, l)
    assert e.value.code == mad.MAD_EINVAL
    with pytest.raises(ValueError, match="head_dim"):
        mad.draft_decode_attn(q, mad.KV(k[..., :32].contiguous(), k[..., :32].contiguous(), as_seq([1, 1])), None, None,
                              None, o, l)
    with pytest.raises(ValueError, match="contiguous"):
        mad.draft_decode_attn(q.transpose(0, 1).contiguous().transpose(0, 1), mad.KV(k, k, as_seq([1, 1])), None, None,
                              None, o, l)
    # a length, or a ring start, too many
    with pytest.raises(IndexError):
        mad.draft_decode_attn(q, mad.KV(k, k, as_seq([1, 1, 1])), None, None, None, o, l)
    with pytest.raises(IndexError):
        mad.draft_decode_attn(q, None, mad.KV(k, k, as_seq([1, 1]), as_seq([0, 0, 0])), None, None, o, l)
    qv, ov, lv = q[:, None].contiguous(), torch.empty(2, 1, 8, 64, dtype=torch.bfloat16, device="cuda"), l[:, None].contiguous()
    with pytest.raises(IndexError):
        mad.verify_attn(qv, mad.KV(k, k, as_seq([1, 1, 1])), ov, lv)


@contextlib.contextmanager
def _entry(mad, name, fn):
    """The native functions call `fn` in place of the C entry point `name` (nothing is enqueued)."""
    lib, fast = mad._load_library(), mad._fast()
    stub = ctypes.CFUNCTYPE(ctypes.c_int, *getattr(lib, name).argtypes)(fn)
    address = lambda n: ctypes.cast(stub if n == name else getattr(lib, n), ctypes.c_void_p).value
    fast.bind(tuple(address(n) for n in mad._FAST_ENTRIES), mad.KV, mad._default_ws, torch._C._cuda_getCurrentRawStream)
    try:
        yield
    finally:
        mad._FAST = None
        mad._fast()


def test_kept_workspace_outlives_its_replacement_during_the_call():
    """The C entry point runs without the interpreter lock, and another thread on the stream may replace the kept
    workspace meanwhile: the old one's memory must not be given back before the entry point has enqueued its work."""
    import paper_2608_30252_amd as mad
    q = torch.zeros(1, 4, 64, dtype=torch.bfloat16, device="cuda")
    kv = mad.KV(torch.zeros(1, 1, 8, 64, dtype=torch.bfloat16, device="cuda"), torch.zeros(1, 1, 8, 64, dtype=torch.bfloat16, device="cuda"), [3])
    o, l = torch.empty_like(q), torch.empty(1, 4, device="cuda")
    mad.draft_decode_attn(q, kv, None, None, None, o, l)   # the workspace of this stream exists from here on
    torch.cuda.synchronize()
    kept = mad._default_ws[(q.device.index, torch.cuda.current_stream().cuda_stream)]
    seen = []

    def replaced(*args):
        old = weakref.ref(kept.buf)
        kept.buf = None
        seen.append(old() is not None)
        return mad.MAD_OK

    with _entry(mad, "mad_draft_decode_attn", replaced):
        mad.draft_decode_attn(q, kv, None, None, None, o, l)
    assert seen == [True]

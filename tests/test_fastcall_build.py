"""Properties of the binding's native module as it is built (no GPU)."""
import os
import struct
import sys
import time

import numpy as np
import pytest
import torch

import paper_2608_30252_amd as mad


def _segment_types(path):
    """p_type of every program header of an ELF64 little-endian file."""
    with open(path, "rb") as f:
        b = f.read()
    assert b[:6] == b"\x7fELF\x02\x01"
    off, = struct.unpack_from("<Q", b, 32)
    size, n = struct.unpack_from("<HH", b, 54)
    return [struct.unpack_from("<I", b, off + i * size)[0] for i in range(n)]


def test_native_module_has_no_thread_local_storage():
    """Loading a library with a thread-local segment slows every access to torch's thread-local variables
    (glibc up to 2.38), and with it each call that the native module does not serve."""
    PT_LOAD, PT_TLS = 1, 7
    types = _segment_types(os.path.join(os.path.dirname(mad.__file__), "_fastcall.so"))
    assert PT_LOAD in types and PT_TLS not in types


def test_without_the_native_module_calls_take_the_ctypes_path(monkeypatch):
    """libmad.so alone serves every call, as it did before there was a native module; a warning says what is missing."""
    monkeypatch.setitem(sys.modules, "paper_2608_30252_amd._fastcall", None)   # an import of it raises
    monkeypatch.delattr(mad, "_fastcall", raising=False)
    monkeypatch.setattr(mad, "_FAST", None)
    w = torch.zeros(64, 64, dtype=torch.bfloat16)
    with pytest.warns(RuntimeWarning, match="_fastcall"):
        assert mad._fast().linear(w, w, w, w) is None
    x = torch.zeros(1, 1, 64)
    with pytest.raises(ValueError, match="w_kv"):   # the ctypes path's own check
        mad.memory_update(x, x[0], [[0]], mad.KV(torch.zeros(1, 1, 8, 64), torch.zeros(1, 1, 8, 64), [0]))


def _us(call, n=500, reps=9):
    best = float("inf")
    for _ in range(reps):
        t = time.perf_counter()
        for _ in range(n):
            assert call() is None
        best = min(best, time.perf_counter() - t)
    return best / n * 1e6


def test_calls_for_the_ctypes_path_go_back_at_once():
    """A call whose argument types send it to the ctypes path must not pay for an attempt: it is told by the types,
    not by an exception half-way (which made such calls 3 - 4 us slower).  Measured against a call that does end by
    an exception: plain arguments whose tensors are not on a GPU."""
    fast = mad._fast()
    bf = lambda *s: torch.zeros(*s, dtype=torch.bfloat16)
    q, o, l, k, x, w = bf(2, 4, 64), bf(2, 4, 64), torch.zeros(2, 4), bf(2, 1, 8, 64), bf(2, 1, 64), bf(128, 64)
    kv = lambda s: mad.KV(k, k, s([1, 2]))
    sub = q.as_subclass(type("Sub", (torch.Tensor,), {}))
    p, u, i32 = torch.zeros(2, 1, 8), torch.zeros(2, 1), torch.zeros(2, dtype=torch.int32)
    qv, ov, lv, xr, gm, plain = q[:, None], o[:, None], l[:, None], x[:, 0], w[0], kv(list)
    thrown = min(_us(lambda: fast.attn(q, plain, None, None, None, o, l, None, None, None)),
                 _us(lambda: fast.verify(qv, plain, ov, lv, None, None)))
    calls = {
        "decode, lengths in an array": lambda a=kv(np.array): fast.attn(q, a, None, None, None, o, l, None, None, None),
        "decode, lengths as array elements": lambda a=kv(lambda s: list(np.array(s))): fast.attn(q, a, None, None, None, o, l, None, None, None),
        "decode, a tensor subclass": lambda a=kv(list): fast.attn(sub, a, None, None, None, o, l, None, None, None),
        "decode, an array scalar as scale": lambda a=kv(list): fast.attn(q, a, None, None, None, o, l, np.float32(1), None, None),
        "step, modes in an array": lambda a=kv(list), m=np.array([1, 1]): fast.attn(q, a, None, q, q, o, l, None, None, m),
        "update, positions in an array": lambda a=kv(list), m=np.array([[1], [2]]): fast.update(x, w, m, a, None, 1e4),
        "update, flags in an array": lambda a=kv(list), m=np.array([1, 0]): fast.update(x, w, [[1], [2]], a, m, 1e4),
        "verify, lengths in an array": lambda a=kv(np.array): fast.verify(qv, a, ov, lv, None, None),
        "stochastic accept without drafts": lambda: fast.stoch(p, None, None, u, i32, i32, None),
        "maps, positions in an array": lambda m=np.array([1, 2]): fast.qkv(xr, gm, w, m, 2, 1, 64, q, q, q, None, 1e-5, 1e4, False),
    }
    for name, call in calls.items():
        t = _us(call)
        assert t < 0.5 * thrown, f"{name}: {t:.2f} us, a call that ends by an exception {thrown:.2f} us"

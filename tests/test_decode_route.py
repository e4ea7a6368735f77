"""The rule that sends a decode launch to the stream kernel or the split kernel (decode_streams), on the CPU.

A slab is 64 keys at head_dim 128 and 128 at 64; a unit is one (sequence, KV head).  The stream kernel
flushes once per unit, so many short units stay with the split kernel, which was the faster one for
them; the shapes here lie on both sides of the rule's lines.
"""
import ctypes

import pytest

from paper_2608_30252_amd.build import LIB

BF16, F32 = 1, 0


def streams(lens, Hkv, G, d, dtype=BF16):
    fn = ctypes.CDLL(LIB)._ZN3mad14decode_streamsEiiiiiPKi
    fn.restype = ctypes.c_bool
    return fn(len(lens), Hkv, G, d, dtype, (ctypes.c_int * len(lens))(*lens))


def ramp(B, lo, hi):
    return [lo + (hi - lo) * b // (B - 1) for b in range(B)]


@pytest.mark.parametrize("lens,Hkv,G,d", [
    ([120] * 64, 8, 1, 128), ([120] * 64, 8, 2, 128), ([120] * 64, 8, 4, 128),   # units of two slabs
    (ramp(64, 50, 256), 8, 4, 128), (ramp(64, 50, 256), 8, 8, 128),             # ragged, 3 slabs a unit
    ([201] * 64, 8, 4, 128), ([257] * 64, 8, 2, 128),                            # even, but their last slabs nearly empty
    ([90] * 64, 8, 8, 64),                                                        # units of one slab
    ([188] * 8, 2, 16, 128),                                                       # few units of 3 slabs
    ([8200], 8, 1, 128),                                                           # one query head per KV head
    ([2200] * 64, 8, 1, 64), (ramp(64, 400, 2048), 8, 1, 64),
])
def test_short_units_and_single_query_heads_stay_with_the_split_kernel(lens, Hkv, G, d):
    assert not streams(lens, Hkv, G, d)


@pytest.mark.parametrize("lens,Hkv,G,d", [
    ([256] * 64, 8, 4, 128), (ramp(64, 148, 778), 8, 4, 128), ([3000] * 4, 8, 4, 128), ([32768], 8, 4, 128),
    ([500] * 16, 8, 8, 64), ([2000], 2, 16, 64), ([3000], 2, 16, 128), ([40] * 16, 2, 16, 128),
    (ramp(64, 600, 3200), 8, 4, 64), ([3000] * 64, 8, 4, 64), (ramp(16, 400, 2048), 8, 2, 128),
])
def test_long_launches_stream(lens, Hkv, G, d):
    assert streams(lens, Hkv, G, d)
    assert not streams(lens, Hkv, G, d, F32)


def test_empty_rows():
    assert not streams([0], 8, 4, 64)
    assert not streams([0] * 64, 8, 4, 128)

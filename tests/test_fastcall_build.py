"""Properties of the binding's native module as it is built (no GPU)."""
import os
import struct

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

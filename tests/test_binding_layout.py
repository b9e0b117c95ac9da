"""The binding hands the library its structs as packed bytes: each field has to lie where the ctypes mirror of the header puts it."""
import ctypes
import struct

from paper_2509_24014_amd import binding


def _fields(cls, raw):
    x = cls.from_buffer_copy(raw)
    return [getattr(x, f[0]) for f in cls._fields_]


def test_packed_structs_match_the_ctypes_mirrors():
    tensor = (0x7fff12345670, 1, 2, 3, 4, 5, 1 << 40, -7, 11)
    index = (1, 2, 3, 4, 32, 64, 2**31 - 1, 0x7fff00000010, 0x7fff00000020)
    execution = (0x10, 0x20, 1 << 41, 0x30, 0x40, 0x50, 0x60)
    for cls, pack, values in ((binding._Tensor, binding._pack_tensor, tensor), (binding._BlockIndex, binding._pack_index, index),
                              (binding._Exec, binding._pack_exec, execution)):
        raw = pack(*values)
        assert len(raw) == ctypes.sizeof(cls)
        assert _fields(cls, raw) == list(values)
    assert struct.calcsize("P") == ctypes.sizeof(ctypes.c_void_p)


def test_null_pointers_are_reported_by_the_byte_entry_points():
    calls = binding._entry()
    zero = binding._pack_tensor(0, 0, 1, 1, 64, 64, 64 * 64, 64 * 64, 64)
    ex = binding._pack_exec(0, 0, 0, 0, 0, 0, 0)
    assert calls.attn_dense(zero, zero, zero, zero, ex) != 0
    assert b"NULL" in binding.load_library().sparsed_last_error()

"""The kernels that hold rows and sums in registers from one transform to the next fit the registers a workgroup of their size
has: what they spill is written and read back in every transform.  Read from the built library's own kernel descriptions."""
import re
import struct

import msgpack
import pytest

from paper_2602_08798_amd import binding

FITS = ("mul_row_kernel", "mul_sum_row_kernel", "ks_row_kernel", "ks_sum_row_kernel", "rot_row_kernel", "ks_wide_kernel", "ks_sum_down_kernel", "ks_unit_kernel")


def _kernels():
    """[(mangled name, registers spilled, scratch bytes per thread)]"""
    lib = open(binding._LIB_PATH, "rb").read()
    at = lib.index(b"__CLANG_OFFLOAD_BUNDLE__")
    count, pos = struct.unpack_from("<Q", lib, at + 24)[0], at + 32
    for _ in range(count):
        offset, size, length = struct.unpack_from("<QQQ", lib, pos)
        target = lib[pos + 24:pos + 24 + length]
        pos += 24 + length
        if b"gfx950" in target:
            obj = lib[at + offset:at + offset + size]
    # the code object's note of type 32 (NT_AMDGPU_METADATA): name and description sizes, type, name padded to 8, description
    note = obj.index(struct.pack("<I", 32) + b"AMDGPU\0\0")
    size = struct.unpack_from("<I", obj, note - 4)[0]
    meta = msgpack.unpackb(obj[note + 12:note + 12 + size])
    return [(k[".name"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in meta["amdhsa.kernels"]]


@pytest.mark.parametrize("family", FITS)
def test_nothing_is_spilled(family):
    mine = [k for k in _kernels() if re.search(rf"\d{family}I", k[0])]
    assert mine
    assert [k for k in mine if k[1] or k[2]] == []

"""Kernels whose waits are counted use no scratch memory (host-only: reads the metadata of the built library).  A reload would wait for
every copy in flight, and the spills of 256 persistent workgroups are traffic of their own."""
import struct

import pytest

from paper_2404_19124_amd import binding as B

msgpack = pytest.importorskip("msgpack")


def kernels():
    """(name, metadata) of every kernel of the library: the notes of its code objects."""
    data = open(B.LIB_PATH, "rb").read()
    at = data.find(b"AMDGPU\0\0")
    while at >= 0:
        name_size, size, kind = struct.unpack_from("<III", data, at - 12)
        if (name_size, kind) == (7, 32):
            for k in msgpack.unpackb(data[at + 8:at + 8 + size])["amdhsa.kernels"]:
                yield k[".name"], k
        at = data.find(b"AMDGPU\0\0", at + 8)


def test_tile_kernel_without_scratch():
    B.lib()
    found = {name: k[".private_segment_fixed_size"] for name, k in kernels() if "head_tile_kernel" in name}
    assert len(found) == 5 and not any(found.values()), found

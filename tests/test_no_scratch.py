"""No kernel of the library keeps registers in scratch memory (a launch with scratch costs 1.5 to 4 us more):
read from the metadata of the code objects in the built library."""
import os
import struct

import pytest

from paper_1912_04822_amd import build

msgpack = pytest.importorskip("msgpack")

EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _kernels(path):
    blob = open(path, "rb").read()
    at = blob.find(b"\x7fELF", 1)
    while at > 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", blob, at + 40)
            size, count = struct.unpack_from("<HH", blob, at + 58)
            for s in range(count):
                _, kind, _, _, off, length = struct.unpack_from("<IIQQQQ", blob, at + shoff + s * size)
                end = off + length
                while kind == SHT_NOTE and off < end:
                    nlen, dlen, note = struct.unpack_from("<III", blob, at + off)
                    data = off + 12 + (nlen + 3) // 4 * 4
                    if note == NT_AMDGPU_METADATA:
                        yield from msgpack.unpackb(blob[at + data:at + data + dlen])["amdhsa.kernels"]
                    off = data + (dlen + 3) // 4 * 4
        at = blob.find(b"\x7fELF", at + 4)


def test_no_kernel_uses_scratch():
    if not os.path.exists(build.LIB):
        build.build_library()
    kernels = list(_kernels(build.LIB))
    assert len({k[".name"] for k in kernels if "backward_kernel" in k[".name"]}) >= 24
    spilled = {k[".name"]: k[".private_segment_fixed_size"] for k in kernels if k[".private_segment_fixed_size"]}
    assert not spilled, spilled

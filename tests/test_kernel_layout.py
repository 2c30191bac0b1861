"""What the kernels' hand-written LDS addresses take for granted, read from the built library's own metadata (no GPU)."""
import struct

import msgpack
import pytest

from paper_2411_18873_amd import eck

EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _kernels(blob):
    """the kernel descriptions of every device image embedded in the library: {name: its fields}"""
    found = {}
    at = blob.find(b"\x7fELF", 1)
    while at > 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == EM_AMDGPU:
            sections, = struct.unpack_from("<Q", blob, at + 40)
            entry, count = struct.unpack_from("<HH", blob, at + 58)
            for s in range(count):
                header = at + sections + s * entry
                offset, = struct.unpack_from("<Q", blob, header + 24)
                if struct.unpack_from("<I", blob, header + 4)[0] != SHT_NOTE:
                    continue
                name_size, size, kind = struct.unpack_from("<III", blob, at + offset)
                data = at + offset + 12 + (name_size + 3) // 4 * 4
                if kind == NT_AMDGPU_METADATA:
                    found.update((k[".name"], k) for k in msgpack.unpackb(blob[data:data + size])["amdhsa.kernels"])
        at = blob.find(b"\x7fELF", at + 1)
    return found


@pytest.fixture(scope="module")
def kernels():
    eck.lib()
    with open(eck.LIB_PATH, "rb") as fh:
        return _kernels(fh.read())


def test_joined_lds_addresses_start_at_zero(kernels):
    """The tree scorer's one-group kernels for bfloat16 features join a row's offset and a lane's place with an OR: the
    dynamic LDS has to start at zero, so the kernels may not declare a __shared__ variable of their own."""
    walks = {n: k for n, k in kernels.items() if "tree_score_kernelILb1" in n and "ELi1EEE" in n}
    assert walks
    for name, k in walks.items():
        assert k[".group_segment_fixed_size"] == 0, name

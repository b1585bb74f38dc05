"""What the built library says of its kernels (the metadata notes of its code objects)."""
import os
import struct

import pytest

import paper_2006_08085_amd as D

msgpack = pytest.importorskip("msgpack")


def _code_objects(blob):
    """The gfx950 code objects of the offload bundles in a shared library, one bundle per source."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", blob, pos - 8)[0]):
            offset, size, length = struct.unpack_from("<QQQ", blob, pos)
            triple = blob[pos + 24:pos + 24 + length]
            pos += 24 + length
            if triple.endswith(b"gfx950"):
                yield blob[at + offset:at + offset + size]
        at += len(magic)


def _kernels():
    if not os.path.exists(D.LIB_PATH):
        from paper_2006_08085_amd.build import build
        build(verbose=False)
    with open(D.LIB_PATH, "rb") as f:
        blob = f.read()
    kernels = {}
    for co in _code_objects(blob):
        at = co.find(b"AMDGPU\0\0")                       # note: name size, description size, type 32, name, description
        size, kind = struct.unpack_from("<II", co, at - 8)
        assert at > 0 and kind == 32
        for k in msgpack.unpackb(co[at + 8:at + 8 + size], strict_map_key=False)["amdhsa.kernels"]:
            kernels[k[".name"]] = k
    return kernels


def test_the_tile_of_the_lds_resident_kernels_starts_at_offset_zero():
    """They address their tile as numbers from 0 on: a static LDS object would lie under it."""
    kernels = _kernels()
    tile = [k for name, k in kernels.items() if "fused_generic" in name]
    assert len(tile) >= 100
    assert {k[".group_segment_fixed_size"] for k in tile} == {0}
    assert any(k[".group_segment_fixed_size"] > 0 for name, k in kernels.items() if "softmax" in name)  # the note is read


def test_so_does_the_tile_of_the_consensus_sequence():
    kernels = [k for name, k in _kernels().items() if "factor_sequence" in name]
    assert len(kernels) >= 6
    assert {k[".group_segment_fixed_size"] for k in kernels} == {0}

"""What the built kernels ask of the hardware, read from the code object in the library: needs no GPU."""
import os
import re
import struct

import msgpack
import pytest


def code_objects(data):
    """The AMD code objects of every offload bundle in an image."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + 24)
        where = at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, where)
            triple = data[where + 24:where + 24 + length]
            where += 24 + length
            if b"gfx950" in triple:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 24)


def kernels_of(elf):
    """The kernel descriptions in the metadata note of a code object."""
    table, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, table + i * size + 4)
        offset, length = struct.unpack_from("<QQ", elf, table + i * size + 24)
        at = offset
        while kind == 7 and at < offset + length:  # notes
            name, desc, note = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3 & ~3)
            if note == 32:  # AMDGPU metadata
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            at = body + (desc + 3 & ~3)


@pytest.fixture(scope="module")
def kernels():
    import paper_1903_00757_amd as gv

    if not os.path.exists(gv.LIB_PATH):
        from paper_1903_00757_amd import build

        build.build()
    with open(gv.LIB_PATH, "rb") as f:
        data = f.read()
    return {k[".name"]: k for elf in code_objects(data) for k in kernels_of(elf)}


def test_waiting_pools_leave_room_for_each_other(kernels):
    """A workgroup of k_train_flow is two waves to each of a compute unit's four SIMDs, which have 512 registers a lane.  Shapes
    of up to 128 registers leave room for a second one, of another context's pool; and all of them keep their rows in
    registers."""
    flow = {tuple(map(int, re.search(r"k_train_flowILi(\d+)ELi(\d+)ELb(\d)ELb(\d)E", name).groups())): k
            for name, k in kernels.items() if "k_train_flowI" in name}
    assert len(flow) == 4 * 5 * 4
    for (V, K, full, track), k in flow.items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, (V, K, full, track)
        if (V, K) in ((1, 1), (1, 2), (2, 1), (2, 2), (4, 1)) or (V, K, track) == (1, 3, 0):
            assert k[".vgpr_count"] <= 128, (V, K, full, track, k[".vgpr_count"])

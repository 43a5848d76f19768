"""What the compiler reports of the built multiply kernels (the metadata of the library's own
code objects): no scalar registers parked in vector lanes, no scratch."""
import re
import struct

import msgpack

import paper_1809_10572_amd as samd


def _code_objects(blob):
    """gfx950 ELF images of the library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", -1
    while (at := blob.find(magic, at + 1)) >= 0:
        entries, p = struct.unpack_from("<Q", blob, at + len(magic))[0], at + len(magic) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + length]:
                yield blob[at + offset:at + offset + size]
            p += 24 + length


def _kernels(elf):
    """The kernel records of an ELF image's AMDGPU metadata note."""
    table, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        _, kind, _, _, p, size = struct.unpack_from("<IIQQQQ", elf, table + i * entry)
        end = p + size
        while kind == 7 and p < end:   # SHT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, p)
            p += 12 + (name + 3) // 4 * 4
            if note == 32:             # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[p:p + desc])["amdhsa.kernels"]
            p += (desc + 3) // 4 * 4


def test_multiply_kernels_keep_their_registers():
    samd.lib()
    with open(samd.LIB_PATH, "rb") as f:
        blob = f.read()
    seen = 0
    for k in (k for elf in _code_objects(blob) for k in _kernels(elf)):
        form = re.search(r"conv2d_samd_kernelILi(\d)ELi(\d)ELi(\d)E", k[".name"])
        if not form:
            continue
        seen += 1
        # one or two values may be parked at an item's start; kernel words never (a batch of them,
        # carried from item to item, was 32 to 100 moves each way)
        assert k[".sgpr_spill_count"] <= 4, k[".name"]
        if int(form[1]) < 4:   # four rows per lane: 64 accumulator registers and more
            assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, k[".name"]
    assert seen == 104

"""What the compiler gave the kernels of the built library, from the metadata beside their code (no GPU)."""
import struct

import msgpack

from .helpers import ensure_built

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(path):
    """The metadata record of every kernel in the library's gfx950 code objects."""
    data = open(path, "rb").read()
    found = []
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, entry)
            name = data[entry + 24:entry + 24 + n]
            entry += 24 + n
            if b"gfx950" in name and size:
                found += notes(data[at + offset:at + offset + size])
        at = data.find(MAGIC, at + 1)
    return found


def notes(elf):
    """amdhsa.kernels of one code object."""
    (start,) = struct.unpack_from("<Q", elf, 32)          # program headers
    size, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        kind, _, offset, _, _, length = struct.unpack_from("<IIQQQQ", elf, start + i * size)
        end = offset + length
        while kind == 4 and offset + 12 <= end:            # notes: name "AMDGPU", type 32: the metadata
            name, desc, what = struct.unpack_from("<III", elf, offset)
            body = offset + 12 + (name + 3) // 4 * 4
            if what == 32 and elf[offset + 12:offset + 18] == b"AMDGPU":
                return msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            offset = body + (desc + 3) // 4 * 4
    return []


def test_medium_batch_kernels_use_no_scratch():
    """Their ring lies in registers: a spilled register is stored and loaded in every step (up to 14 % of the kernel)."""
    found = {k[".name"]: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in kernels(ensure_built().LIB_PATH) if "midm_kernel" in k[".name"]}
    assert len(found) == 11   # nibbles in groups of 128 and bytes with one to four blocks of 16 rows, groups of 64 with up to three
    assert set(found.values()) == {(0, 0)}, found

"""What the compiler gave the kernels, from the metadata in the built library."""
import os
import struct

import msgpack

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2211_17192_amd", "libsd.so")


def kernels():
    """name -> metadata of every kernel: the note of the gfx950 code object in the library's offload bundle."""
    with open(LIB, "rb") as f:
        data = f.read()
    start = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    at, elf = start + 32, None
    for _ in range(struct.unpack_from("<Q", data, start + 24)[0]):
        offset, size, length = struct.unpack_from("<QQQ", data, at)
        if b"gfx950" in data[at + 24:at + 24 + length]:
            elf = data[start + offset:start + offset + size]
        at += 24 + length
    sections, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        _, kind, _, _, offset, _ = struct.unpack_from("<IIQQQQ", elf, sections + i * entry)
        if kind != 7:                                          # SHT_NOTE
            continue
        name, desc, note = struct.unpack_from("<III", elf, offset)
        if note == 32:                                         # NT_AMDGPU_METADATA
            d = offset + 12 + (name + 3) // 4 * 4
            return {k[".name"]: k for k in msgpack.unpackb(elf[d:d + desc])["amdhsa.kernels"]}
    raise AssertionError("no kernel metadata")


def test_products_of_k_slices_use_no_scratch():
    """Chains of launches of a few microseconds each: a register kept in memory is a trip there and back."""
    slices = {n: k[".private_segment_fixed_size"] for n, k in kernels().items() if "gemm_slices_kernel" in n}
    assert len(slices) > 50 and not any(slices.values()), {n: v for n, v in slices.items() if v}

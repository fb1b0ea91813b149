"""The kernels for small products, as built: no instantiation spills registers (a complex patch's four products, and the elements kept for the check of
the slice count, have to fit them at every slice count)."""
import struct

import msgpack

from paper_2306_11975_amd import build


def kernels_of(path):
    """The AMDGPU metadata of every gfx950 kernel in a shared library built here, by mangled name."""
    raw, at, found = path.read_bytes(), 0, {}
    while (at := raw.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entries, p = struct.unpack_from("<Q", raw, at + 24)[0], at + 32
        for _ in range(entries if entries < 8 else 0):
            offset, size, length = struct.unpack_from("<QQQ", raw, p)
            target, p = raw[p + 24:p + 24 + length], p + 24 + length
            if b"gfx950" not in target or size == 0:
                continue
            elf = raw[at + offset:at + offset + size]
            sections, = struct.unpack_from("<Q", elf, 40)
            entry_size, count = struct.unpack_from("<HH", elf, 58)
            for i in range(count):
                kind, = struct.unpack_from("<I", elf, sections + i * entry_size + 4)
                start, = struct.unpack_from("<Q", elf, sections + i * entry_size + 24)
                if kind == 7:   # SHT_NOTE
                    name, desc, _ = struct.unpack_from("<III", elf, start)
                    data = elf[start + 12 + (name + 3) // 4 * 4:][:desc]
                    found.update({k[".name"]: k for k in msgpack.unpackb(data)["amdhsa.kernels"]})
        at += 24
    return found


def test_small_kernels_do_not_spill():
    small = {n: k for n, k in kernels_of(build.LIB).items() if "small_product_kernel" in n or "small_complex_kernel" in n}
    assert len(small) > 60
    spilling = {n: k[".vgpr_spill_count"] for n, k in small.items() if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilling, spilling

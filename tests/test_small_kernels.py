"""The kernels for small products on the host: no instantiation spills registers (a complex patch's four products, and the elements kept for the check of
the slice count, have to fit them at every slice count), and the rules that choose them keep to the sizes where they take less than two launches."""
import ctypes
import struct

import msgpack
import pytest

from paper_2306_11975_amd import build
from paper_2306_11975_amd import ozimmu


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


def rule(symbol, *types):
    f = getattr(ozimmu.lib(), symbol)
    f.restype, f.argtypes = ctypes.c_bool, types
    return f


I64, PTR = ctypes.c_int64, ctypes.c_void_p
COMPLEX_AHEAD = "_ZN6ozimmu19small_complex_aheadEPKdS1_S1_llli"


@pytest.mark.parametrize("m,n,k,s,ahead", [(8192, 2, 2, 11, True), (8192, 2, 2, 12, False), (300, 16, 16, 16, False), (300, 17, 16, 16, True), (2000, 16, 64, 13, False),
                                           (4096, 64, 16, 16, True), (1, 1, 1, 12, False), (8225, 2, 2, 3, False)])
def test_narrow_gates_of_many_slices_are_left_to_the_gate_kernel(m, n, k, s, ahead):
    f = rule(COMPLEX_AHEAD, PTR, PTR, PTR, I64, I64, I64, ctypes.c_int)
    assert f(256, 512, 1024, m, n, k, s) == ahead
    # operands that the gate kernel does not take (8 bytes off a complex element's alignment) have only the general path otherwise
    assert f(256, 512, 1032, m, n, k, s) == (m <= 8192)


# 32 x 32 tiles times steps of 64 positions: four to a compute unit, fewer where two launches take less
@pytest.mark.parametrize("m,n,k,s,by_rows,applies", [
    (1024, 1024, 64, 8, False, True), (1025, 1024, 64, 8, False, False), (512, 1024, 128, 16, False, True), (512, 1024, 129, 8, False, False),
    (256, 1024, 256, 8, False, True), (256, 1024, 256, 9, False, False),
    # both operands along k, at one step: three, but four with ten to thirteen slices
    (768, 1024, 64, 9, True, True), (769, 1024, 64, 9, True, False), (1024, 1024, 64, 10, True, True), (1024, 1024, 64, 13, True, True), (769, 1024, 64, 14, True, False),
    (512, 1024, 128, 9, True, True), (256, 1024, 256, 3, True, True),
    # half a step with more than nine slices
    (1024, 1024, 32, 13, False, True), (1024, 1024, 32, 14, False, False), (768, 1024, 32, 16, False, True), (1024, 1024, 33, 16, False, True),
    (769, 1024, 32, 10, True, False), (768, 1024, 32, 13, True, True), (513, 1024, 32, 14, True, False), (512, 1024, 32, 16, True, True)])
def test_limits_of_the_small_product(m, n, k, s, by_rows, applies):
    f = rule("_ZN6ozimmu21small_product_appliesElllib", I64, I64, I64, ctypes.c_int, ctypes.c_bool)
    assert f(m, n, k, s, by_rows) == applies


def test_counters_of_every_size_fit_their_buffer():
    """8192 words behind the sums (the larger of what the small kernels and the splitter leave): two per plane and tile of rows or columns of 32."""
    real = rule("_ZN6ozimmu21small_product_appliesElllib", I64, I64, I64, ctypes.c_int, ctypes.c_bool)
    cplx = rule("_ZN6ozimmu21small_complex_appliesEllli", I64, I64, I64, ctypes.c_int)
    largest = 0
    for tiles_m in [*range(1, 70), *range(70, 2100, 13), 1023, 1024, 1025]:
        for tiles_n in (1, 2, 3, 7, 16, 31, 32, 33, 256, 257, 1024, 1025):
            for a, b in ((tiles_m, tiles_n), (tiles_n, tiles_m)):
                for planes, takes in ((1, real(32 * a, 32 * b, 1, 3, False)), (2, cplx(32 * a, 32 * b, 1, 3))):
                    if takes:
                        largest = max(largest, 2 * planes * (a + b))
    assert 2050 <= largest <= 8192

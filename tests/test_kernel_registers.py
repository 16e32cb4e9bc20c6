"""Registers of the built kernels, read from the code objects' own metadata.  A spilled register in a transform, a rescale or
a MAC loop is a wait for memory in the middle of it, which no test of the results would show."""
import re
import struct

import msgpack
import pytest

from paper_1908_04172_amd import he


def code_objects(data):
    """The gfx950 code objects in the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        entries, pos = struct.unpack_from("<Q", data, at + len(magic))[0], at + len(magic) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + length] and size:
                yield data[at + offset:at + offset + size]
            pos += 24 + length
        at = data.find(magic, at + len(magic))


def kernels():
    found = {}
    for elf in code_objects(open(he.LIB_PATH, "rb").read()):
        sections, entry, count = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
        for k in range(count):
            kind, offset, size = (struct.unpack_from("<I", elf, sections + k * entry + 4)[0],
                                  *struct.unpack_from("<QQ", elf, sections + k * entry + 24))
            if kind != 7:  # a note section: (name size, descriptor size, type), name, descriptor
                continue
            name, desc, note = struct.unpack_from("<III", elf, offset)
            if note == 32:  # AMDGPU metadata
                start = offset + 12 + (name + 3) // 4 * 4
                for kernel in msgpack.unpackb(elf[start:start + desc])["amdhsa.kernels"]:
                    found[kernel[".name"]] = kernel
    return found


@pytest.fixture(scope="module")
def built():
    return kernels()


def matching(built, pattern):
    names = {n: k for n, k in built.items() if re.search(pattern, n)}
    assert names, pattern
    return names


def test_rescale_kernels_do_not_spill(built):
    found = matching(built, r"\d+(scaled_)?rescale_kernel")
    assert len(found) == 10                                     # two per ring degree, whether a polynomial is split or not
    for name, k in found.items():
        assert k[".vgpr_spill_count"] == 0 and k[".vgpr_count"] <= 128, (name, k[".vgpr_count"], k[".vgpr_spill_count"])


@pytest.mark.parametrize("pattern,registers", [(r"ntt_rows_kernel", 128), (r"ntt32_rows_kernel", 128), (r"rescale32_kernel", 128),
                                               (r"mac_digits", 256), (r"mac_poly_kernel", 256), (r"key_product_kernel", 256),
                                               (r"encode_vector_kernel", 128)])
def test_other_kernels_do_not_spill(built, pattern, registers):
    """... and stay within what their wavefronts per SIMD leave them (512 registers per lane)."""
    for name, k in matching(built, pattern).items():
        assert k[".vgpr_spill_count"] == 0 and k[".vgpr_count"] <= registers, (name, k[".vgpr_count"], k[".vgpr_spill_count"])


def test_launches_of_several_classes_keep_to_their_scalar_registers(built):
    """What only launches of one class choose between stays out of their three branches: it is parked in lanes of vector registers and
    fetched back in the loop over the terms (146, 118 and 79 of them cost launches of two classes 2 %)."""
    for pattern, most in ((r"mac_digits_mixed_kernelImLb0E", 110), (r"mac_digits_mixed_kernelImLb1E", 75), (r"mac_digits_mixed_kernelIjLb0E", 48)):
        for name, k in matching(built, pattern).items():
            assert k[".sgpr_spill_count"] <= most, (name, k[".sgpr_spill_count"])

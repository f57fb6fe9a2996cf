"""What the compiler made of the kernels, from the metadata of the code objects in the built library: no kernel
keeps its operands in scratch memory, where every load would be waited for and written back."""
import re
import struct

import msgpack
import pytest

from paper_2309_06626_amd import binding as B

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels_of(elf):
    """Kernel descriptions in the AMDGPU metadata note of a code object (little-endian ELF64)."""
    sections, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        _, kind, _, _, at, length = struct.unpack_from("<IIQQQQ", elf, sections + i * size)
        end = at + length
        while kind == 7 and at < end:  # SHT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if note == 32:  # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[body: body + desc])["amdhsa.kernels"]
            at = body + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    found = {}
    at = data.find(BUNDLE)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(entries):
            offset, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24: p + 24 + name]:
                for k in kernels_of(data[at + offset: at + offset + size]):
                    found[k[".name"]] = k
            p += 24 + name
        at = data.find(BUNDLE, at + 24)
    return found


# bytes a lane that have always been there: spilled registers of the streaming band kernel's widest form, which no automatic choice
# takes, and eight of the depthwise kernel that looks up the rows of its compact input
SPILLS = {"bandstream_kernel": 112, "depthwise3x3_dot2_kernel": 36}


def test_no_kernel_works_in_scratch_memory(kernels):
    assert len(kernels) > 300
    assert sum("igemm_stage_kernel" in n for n in kernels) >= 70
    for name, k in kernels.items():
        plain = re.match(r"_ZN2sc\d+(\w+?_kernel)", name)
        allowed = SPILLS.get(plain.group(1), 0) if plain else 0
        assert k[".private_segment_fixed_size"] <= allowed, (name, k[".private_segment_fixed_size"])


def test_four_row_panel_wavefronts_fit_a_simd(kernels):
    """A row panel of one K tile leaves LDS for four workgroups of four wavefronts; the 512 registers of a SIMD have to as well."""
    panels = [k[".vgpr_count"] for n, k in kernels.items() if "igemm_panel_kernel" in n]
    assert len(panels) == 2 and max(panels) <= 128

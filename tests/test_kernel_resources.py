"""What the compiler gave the kernels of the built library, read from the code objects' own metadata: no kernel keeps
vector registers in memory.  (A spill inside a loop over tiles costs more than the loads it stands beside, and a build
says nothing about it.)  No GPU."""
import re
import struct

import pytest

from paper_2209_02882_amd import binding

msgpack = pytest.importorskip("msgpack")  # the metadata's encoding
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def notes(elf):
    """(type, description) of every note of an ELF64 image that starts at elf[0]."""
    section_table, = struct.unpack_from("<Q", elf, 40)
    sections, = struct.unpack_from("<H", elf, 60)
    for i in range(sections):
        kind, = struct.unpack_from("<I", elf, section_table + 64 * i + 4)
        if kind != SHT_NOTE:
            continue
        at, size = struct.unpack_from("<QQ", elf, section_table + 64 * i + 24)
        end = at + size
        while at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            yield note, elf[at:at + desc]
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """Metadata of every kernel: the code objects lie one after the other inside the library."""
    data = memoryview(open(binding.LIB_PATH, "rb").read())
    raw, found, at = data.obj, [], 0
    while (at := raw.find(b"\x7fELF\x02", at)) >= 0:
        if len(raw) - at > 64 and struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            for note, desc in notes(data[at:]):
                if note == NT_AMDGPU_METADATA:
                    found += msgpack.unpackb(desc, strict_map_key=False)["amdhsa.kernels"]
        at += 4
    assert len(found) > 1000
    return found


# instances with two registers in memory, faster than the forms without (beside the kernel in sgap_sddmm.hip)
KNOWN = {f"sddmm_tile_kernelILi{g}ELi4ELb1ELi2E": 2 for g in (2, 4, 8, 16, 32)}


def test_no_vector_register_is_spilled(kernels):
    spilled = {k[".name"]: k[".vgpr_spill_count"] for k in kernels if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not {name: n for name, n in spilled.items() if n > max([0] + [KNOWN[part] for part in KNOWN if part in name])}


def test_scalar_registers_leave_the_wavefronts_that_a_persistent_grid_counts_on(kernels):
    """sddmm_tile_kernel's grid is what the runtime says is resident at once, which goes by the vector registers (512 per lane of a
    SIMD, in eights).  A SIMD has 800 scalar ones, in sixteens, and the trap handler takes sixteen of each wavefront."""
    quads = [k for k in kernels if re.search(r"sddmm_tile_kernelILi\d+ELi\dELb0ELi1ELb1EE", k[".name"])]  # entries in step, looks for quads
    assert len(quads) == 6
    for k in quads:
        by_vector = 512 // (-(-k[".vgpr_count"] // 8) * 8)
        by_scalar = 800 // (-(-k[".sgpr_count"] // 16) * 16 + 16)
        assert by_scalar >= by_vector, (k[".name"], k[".vgpr_count"], k[".sgpr_count"])

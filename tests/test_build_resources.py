"""Registers of the compiled kernels, from the metadata that the compiler writes into the
library (amdhsa.kernels in the code object's notes): what the sources say about them."""
import os
import struct

import pytest

from paper_1912_05529_amd import mig

msgpack = pytest.importorskip("msgpack")

AMDGPU, SHT_NOTE, NT_METADATA = 224, 7, 32


def _code_objects(blob):
    at = blob.find(b"\x7fELF")
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == AMDGPU:
            yield blob[at:]
        at = blob.find(b"\x7fELF", at + 4)


def _kernels(elf):
    table = struct.unpack_from("<Q", elf, 40)[0]
    size, count = struct.unpack_from("<HH", elf, 58)
    for header in (table + i * size for i in range(count)):
        if struct.unpack_from("<I", elf, header + 4)[0] != SHT_NOTE:
            continue
        note = struct.unpack_from("<Q", elf, header + 24)[0]
        name, desc, kind = struct.unpack_from("<III", elf, note)
        if kind == NT_METADATA:
            at = note + 12 + (name + 3) // 4 * 4
            yield from msgpack.unpackb(elf[at:at + desc], strict_map_key=False)["amdhsa.kernels"]


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(mig.LIB_PATH):
        from paper_1912_05529_amd import build
        build.build_lib()
    with open(mig.LIB_PATH, "rb") as f:
        blob = f.read()
    found = [k for elf in _code_objects(blob) for k in _kernels(elf)]
    assert found
    return found


def _named(kernels, name):
    # mangled names: the length of the identifier, then the identifier
    part = "%d%s" % (len(name), name)
    picked = [k for k in kernels if part in k[".name"]]
    assert picked, name
    return picked


def test_design_keeps_to_vector_registers(kernels):
    """No accumulation registers, spills or scratch in any instance of the table design."""
    for k in _named(kernels, "k_design"):
        got = (k.get(".agpr_count", 0), k[".vgpr_spill_count"], k[".private_segment_fixed_size"])
        assert got == (0, 0, 0), (k[".name"], got)
        assert k[".vgpr_count"] <= 256, k[".name"]

"""No kernel of the built library keeps vector registers in memory: a spilled
row or accumulator is re-read on every use, which no timing of the library
assumes.  Read from the metadata notes of the library's own code objects."""
import struct

import pytest

from paper_2511_05814_amd import binding as b

msgpack = pytest.importorskip("msgpack")

EM_AMDGPU, PT_NOTE, NT_AMDGPU_METADATA = 224, 4, 32


def kernels():
    b.lib()  # says what to do when nothing is built
    data = open(b.LIB_PATH, "rb").read()
    found = []
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            phoff, = struct.unpack_from("<Q", data, at + 32)
            phentsize, phnum = struct.unpack_from("<HH", data, at + 54)
            for i in range(phnum):
                kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + i * phentsize)
                pos, end = at + off, at + off + size
                while kind == PT_NOTE and pos + 12 <= end:
                    nsz, dsz, typ = struct.unpack_from("<III", data, pos)
                    body = pos + 12 + (nsz + 3) // 4 * 4
                    if typ == NT_AMDGPU_METADATA and data[pos + 12:pos + 18] == b"AMDGPU":
                        found += msgpack.unpackb(data[body:body + dsz])["amdhsa.kernels"]
                    pos = body + (dsz + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 1)
    return found


def test_no_kernel_spills_vector_registers():
    ks = kernels()
    names = [k[".name"] for k in ks]
    for part in ("prefill_route_plan_kernel", "prefill_gemm_kernel", "router_kernel", "ffn_down_wide_kernel"):
        assert any(part in n for n in names), part
    spilled = {k[".name"]: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in ks
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled

"""CPU check of the registers of the library's kernels, from the notes that the compiler
writes next to each of them: kernels that are documented to hold everything in
registers spill none of it to scratch memory."""

import re
import struct

import msgpack
import pytest

from paper_2103_14890_amd import qcoll


def _kernels():
    """Metadata of every kernel in the library, by mangled name."""
    data, out = open(qcoll.LIB_PATH, "rb").read(), {}
    for m in re.finditer(re.escape(b"AMDGPU\0\0"), data):   # note: name size, content size, type, name, content
        name_size, size, kind = struct.unpack_from("<3I", data, m.start() - 12)
        if name_size != 7 or kind != 32 or m.end() + size > len(data):   # NT_AMDGPU_METADATA
            continue
        for k in msgpack.unpackb(data[m.end():m.end() + size])["amdhsa.kernels"]:
            out[k[".name"]] = k
    return out


# the batched kernel: Lb0E for launches of matrix slots alone, Lb1E with FFT slots (not held here)
@pytest.mark.parametrize("name", ["multi_kernelILb0E", "fx16_t16", "fp32_t16", "fx16_t32", "fp32_t32", "fx16_t64",
                                  "fp32_t64", "galerkin"])
def test_kernels_without_spills(name):
    kernels = [k for n, k in _kernels().items() if name in n]
    assert kernels, name
    for k in kernels:
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, k[".name"]


@pytest.mark.parametrize("name", ["fx16_t16_kernelILi%dEEE", "fp32_t16_kernelILi%dEEE", "fx16_t32_kernelILi%dELi16EEE",
                                  "fp32_t32_kernelILi%dELi12EEE", "fp32_t32_kernelILi%dELi16EEE"])
def test_projection_holds_no_table_in_lane_registers(name):
    """The 16 entries of the inverse Gram matrix (32 registers) stay out of the lanes'
    registers: the kernel with the projection has about as many as the one without."""
    regs = {n: k[".vgpr_count"] for n, k in _kernels().items()}
    plain, proj = (next(v for n, v in regs.items() if name % kind in n) for kind in (0, 1))
    assert proj <= plain + 12

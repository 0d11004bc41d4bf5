"""Register spills of the library's kernels, from the metadata that the
compiler stores with each kernel of libclamp.so: vector registers that go to
scratch memory cost the bandwidth-bound passes time that no other test
shows."""

import re

import msgpack

from helpers import LIB

# the kernel descriptions: an ELF note "AMDGPU" of type 32 holding a msgpack map
NOTE = re.compile(rb"\x07\x00\x00\x00(....)\x20\x00\x00\x00AMDGPU\x00\x00", re.S)


def kernels():
    data = open(LIB, "rb").read()
    out = {}
    for m in NOTE.finditer(data):
        size = int.from_bytes(m.group(1), "little")
        for k in msgpack.unpackb(data[m.end():m.end() + size])["amdhsa.kernels"]:
            out[k[".name"]] = k
    return out


def test_no_kernel_spills_vector_registers():
    ks = kernels()
    assert any("k_row_grad" in n for n in ks) and any("k_conv" in n for n in ks)
    spilled = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in ks.items()
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled

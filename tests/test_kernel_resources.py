"""Register use of the built kernels, from the notes of the code objects in
libdq.so: none of them spills."""
import struct

import msgpack

import paper_2609_26333_amd as dq


def kernels():
    raw = open(dq.LIB_PATH, "rb").read()
    at = 0
    while True:   # ELF notes: name size, descriptor size, type, "AMDGPU", descriptor
        at = raw.find(b"AMDGPU\0\0", at)
        if at < 0:
            return
        name, desc, kind = struct.unpack_from("<III", raw, at - 12)
        if name == 7 and kind == 32 and at + 8 + desc <= len(raw):
            yield from msgpack.unpackb(raw[at + 8:at + 8 + desc])["amdhsa.kernels"]
        at += 8


def test_no_kernel_spills():
    seen = {k[".name"]: k for k in kernels()}
    assert len(seen) > 100 and any("lut_gemv_batch_kernelILi4ELi2ELi3ELi16E" in n for n in seen)
    bad = {n: (k[".vgpr_count"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in seen.items()
           if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not bad, bad

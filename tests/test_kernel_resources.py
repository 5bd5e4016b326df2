"""Register use of the built kernels, from the notes of the code objects in
libdq.so: none of them spills, and as many workgroups fit on a compute unit as
the plans assume."""
import re
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


def test_short_gemm_residency():
    """The short-grid GEMM kernels leave room for the two workgroups per compute
    unit that the choice of the 32 x 32, 32 x 64, 96 x 64 and 64 x 96 tiles
    assumes: 512 registers per SIMD lane over the wavefronts of a SIMD."""
    seen = 0
    for k in kernels():
        m = re.search(r"nvfp4_gemm_short_kernel.*?ShortGeoILi(\d)ELi(\d)ELi(\d)E", k[".name"])
        if m:
            tm, tn, waves = map(int, m.groups())
            conc = 2 if (tm, tn) in ((1, 1), (1, 2), (3, 2), (2, 3)) else 1
            regs = (k[".vgpr_count"] + 7) // 8 * 8
            assert 512 // regs >= conc * waves // 4, (k[".name"], regs)
            seen += 1
    assert seen == 36

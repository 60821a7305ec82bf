"""Registers and LDS of the built kernels: every item kernel fits a compute unit as many
times as the planner counts on (item sizes, the tail taper and the persistent batch grid,
which must not start more workgroups than can run at once). Read from the kernel metadata
in the library: four workgroups of FP32 taps by moments, three of table taps, 24 of one
wave, per compute unit of 160 KB of LDS and 512 registers per lane and SIMD."""
import re
import struct

import msgpack

from paper_1810_11359_amd import ism


def kernels():
    """Metadata of every gfx950 kernel in the library, by name."""
    data = open(ism.LIB_PATH, "rb").read()
    out = {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:  # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", data, at + 32)
            phnum, = struct.unpack_from("<H", data, at + 56)
            for i in range(phnum):
                ptype, _, off, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + 56 * i)
                if ptype != 4:  # PT_NOTE
                    continue
                p, end = at + off, at + off + size
                while p + 12 <= end:
                    nlen, dlen, kind = struct.unpack_from("<III", data, p)
                    p += 12 + (nlen + 3) // 4 * 4
                    if kind == 32:  # NT_AMDGPU_METADATA
                        for k in msgpack.unpackb(data[p:p + dlen])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    p += (dlen + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 1)
    return out


def test_item_kernels_fit_as_often_as_planned():
    checked = 0
    for name, k in kernels().items():
        # <WT, TL, KIND (moments, FP16, one wave), LUT, POLAR, GEN>
        m = re.search(r"accumulate_(?:batch_)?kernelILi\d+ELi\d+ELi([012])ELb([01])ELb[01]ELb[01]E", name)
        if not m or m[1] == "1":
            continue
        waves = 6 if m[1] == "2" else 3 if m[2] == "1" else 4  # per SIMD
        threads = 64 if m[1] == "2" else 256
        groups = waves * 4 * 64 // threads  # per compute unit
        assert k[".max_flat_workgroup_size"] == threads, name
        assert k[".group_segment_fixed_size"] * groups <= 160 * 1024, (name, k[".group_segment_fixed_size"])
        regs = -(-k[".vgpr_count"] // 8) * 8  # of both kinds, one file
        assert regs * waves <= 512, (name, regs)
        checked += 1
    # moments, FP32: 12 windows x two tiles x directional or not; table taps: 4 windows; one
    # wave: 12 and 4; single and batch
    assert checked == 2 * (12 * 4 + 4 * 2 + 12 * 2 + 4 * 2)

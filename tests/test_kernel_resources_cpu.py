"""Registers of the built kernels, read from the code objects in libdisco.so (their own metadata notes; no GPU).

A compute unit has 512 vector registers per SIMD lane and a workgroup of eight wavefronts puts two on every SIMD: up to 128
registers two workgroups are resident, and a launch of more than 256 workgroups overlaps one's tail with the other's stream."""
import re
import struct

import msgpack

from paper_2405_04304_amd import binding as B


def _kernels():
    """{mangled name: metadata} of every gfx950 kernel in the library."""
    raw, out, at = open(B.LIB_PATH, "rb").read(), {}, 0
    while (at := raw.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        n, p = struct.unpack_from("<Q", raw, at + 24)[0], at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", raw, p)
            if size and b"gfx950" in raw[p + 24:p + 24 + length]:
                out.update(_notes(raw[at + off:at + off + size]))
            p += 24 + length
        at += 24
    return out


def _notes(elf):
    table, (entry, count), out = struct.unpack_from("<Q", elf, 40)[0], struct.unpack_from("<HH", elf, 58), {}
    for i in range(count):
        kind = struct.unpack_from("<I", elf, table + i * entry + 4)[0]
        at, size = struct.unpack_from("<QQ", elf, table + i * entry + 24)
        end = at + size
        while kind == 7 and at < end:                     # a section of notes
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if note == 32:                                # the kernels' metadata
                out.update({k[".name"]: k for k in msgpack.unpackb(elf[at:at + desc], raw=False)["amdhsa.kernels"]})
            at += (desc + 3) // 4 * 4
    return out


def test_deferred_layernorm_costs_no_resident_workgroup():
    gemm = {}
    for name, k in _kernels().items():
        m = re.match(r"_ZN5disco6k_gemmILi(\d+)ELi(\d+)ELi(\d+)ELi8ELi(\d+)ELb([01])E", name)
        if m:
            assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name
            waves = 512 // (-(-k[".vgpr_count"] // 8) * 8)
            gemm[m.groups()] = (min(waves // 2, 2), k[".vgpr_count"])
    layernorm = [key for key in gemm if key[4] == "1"]
    assert len(layernorm) >= 25
    for key in layernorm:
        plain = key[:4] + ("0",)
        assert gemm[key][0] == gemm[plain][0], (key, gemm[key], gemm[plain])

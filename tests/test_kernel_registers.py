"""Registers of the built kernels, from the notes of the gfx950 code objects in
libkmip.so (CPU only)."""
import os
import re
import struct
import subprocess

import paper_2604_03815_amd.build as kbuild

READELF = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(kbuild.HIPCC))), "lib", "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernel_figures(tmp_path):
    """{kernel symbol: {".vgpr_spill_count": n, ".private_segment_fixed_size": n, ..}}"""
    if not os.path.exists(kbuild.LIB):
        kbuild.build()
    data = open(kbuild.LIB, "rb").read()
    found, at = {}, data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" not in name or size == 0:
                continue
            obj = tmp_path / "obj.co"
            obj.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
            for part in re.split(r"\n  - \.", notes)[1:]:
                sym = re.search(r"\.name:\s+(_Z\S+)", part)
                if sym:
                    found[sym.group(1)] = {m[0]: int(m[1]) for m in re.findall(r"(\.\w+):\s+(\d+)\n", part)}
        at = data.find(MAGIC, pos)
    return found


def test_coefficient_pass_keeps_its_registers(tmp_path):
    # A launch bound of four waves per SIMD is for the widths at which it costs
    # next to no registers: 45 spilled ones (152 bytes of scratch a lane) cost
    # a fifth of the backward at d = 32, d_V = 64, k = 16.
    coef = {s: f for s, f in kernel_figures(tmp_path).items() if "coef_split_kernel" in s}
    assert len(coef) == 88   # 3 x 4 widths of 6 slot counts, and d = 128 of 4
    spilled = {s: (f[".vgpr_spill_count"], f[".private_segment_fixed_size"]) for s, f in coef.items()}
    assert {s: x for s, x in spilled.items() if x[0] > 8 or x[1] > 32} == {}

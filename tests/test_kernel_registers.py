"""Registers of the built kernels, from the code object's metadata (no GPU needed): where LDS lets a CU hold more
workgroups than another path of a shared kernel would in registers."""
import os
import re
import struct
import subprocess

import pytest

from paper_2605_08123_amd.build import LIB

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def kernel_registers(tmp_path):
    """{mangled kernel name: VGPRs} of the gfx950 code object inside the library."""
    blob = open(LIB, "rb").read()
    at = blob.find(BUNDLE)
    assert at >= 0, "no offload bundle in the library"
    pos, n = at + len(BUNDLE) + 8, struct.unpack_from("<Q", blob, at + len(BUNDLE))[0]
    for _ in range(n):
        off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
        ident = blob[pos + 24:pos + 24 + idlen].decode()
        pos += 24 + idlen
        if "gfx950" in ident:
            obj = tmp_path / "device.o"
            obj.write_bytes(blob[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
            return {m.group(1): int(m.group(2))
                    for m in re.finditer(r"\.name: +(_Z\S+vsweep_kernel\S+).*?\.vgpr_count: +(\d+)", notes, re.S)}
    pytest.fail("no gfx950 code object in the library")


@pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(READELF), reason="library not built, or no llvm-readelf")
def test_half_steps_at_d32_keep_the_wavefronts_that_lds_allows(tmp_path):
    """bf16, d = 32: rings of 21.5 KB, seven workgroups (wavefronts per SIMD) in 160 KB of LDS; 512 registers per lane and
    SIMD in blocks of eight are 72 for seven wavefronts, 80 for six (256-row blocks).  The dustbin element, which
    is part of the same kernel, must not take more."""
    regs = kernel_registers(tmp_path)
    for mode in (0, 1):   # first half-step, half-step
        for fr, limit in ((1, 72), (2, 80)):
            least = min(v for k, v in regs.items() if re.search(rf"IDF16bLi32ELi{mode}ELi{fr}E", k))
            assert least <= limit, (mode, fr, least)

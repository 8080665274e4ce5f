"""Registers and scratch of kernels whose speed depends on them, as the built library's metadata states them."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2406_02542_amd.build import LIB_PATH

READELF = next((p for p in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf")) if p and os.path.exists(p)), None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled-ish symbol: (registers, scratch bytes)} of every kernel in the library."""
    if READELF is None or not os.path.exists(LIB_PATH):
        pytest.skip("needs the built library and llvm-readelf")
    blob, found, at = open(LIB_PATH, "rb").read(), {}, 0
    out = tmp_path_factory.mktemp("objects")
    while (at := blob.find(MAGIC, at)) >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n if n < 16 else 0):  # (offset, size, length of the target's name, name)
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" not in target or size == 0:
                continue
            path = out / f"{at}.co"
            path.write_bytes(blob[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for block in notes.split("- .agpr_count:")[1:]:
                def field(key):
                    return re.search(rf"\.{key}:\s+(\S+)", block)[1]
                found[field("name")] = (int(field("vgpr_count")), int(field("private_segment_fixed_size")))
        at += len(MAGIC)
    return found


def test_tridiagonalisation_of_more_heads_than_cus_shares_a_cu(kernels):
    """Two blocks of 4 waves on the 4 SIMDs of a CU: at most 256 of a SIMD's 512 registers each, nothing in scratch."""
    (regs, scratch), = [v for k, v in kernels.items() if "tridiag_kernelILi2E" in k]
    assert regs <= 256 and scratch == 0


def test_selection_and_attention_in_one_launch_keep_their_registers(kernels):
    """A list that grows is completed in one place, whatever the form of the loads around it: nothing in scratch, and with
    one head per block room for four waves a SIMD."""
    found = {k: v for k, v in kernels.items() if "select_attend_kernel" in k}
    assert found
    for name, (regs, scratch) in found.items():
        assert scratch == 0, name
        if "BF16ELi1E" in name or "F32ELi1E" in name:
            assert regs <= 128, name

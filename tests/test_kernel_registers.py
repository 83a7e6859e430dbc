"""Registers that the attention kernels keep in scratch memory, from the notes of the built library.  A reload inside a tile loop waits
for every load in flight, the next tiles among them (the dQ kernel at d = 128 with six such reloads a tested tile: 32 x 8192 rows in
128 buckets 489 us a step against 466).  One register of it is kept there across all loops, which costs nothing."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2306_01160_amd import binding

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
ALLOWED = {"attn_bwd_dq_f16_kernelILi128E": 1}


def _spilled(tmp_path):
    lib = open(binding.LIB_PATH, "rb").read()
    out, at = {}, lib.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", lib, at + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", lib, entry)
            if b"gfx950" in lib[entry + 24:entry + 24 + length]:
                (tmp_path / "object").write_bytes(lib[at + offset:at + offset + size])
                notes = subprocess.run([READELF, "--notes", str(tmp_path / "object")], capture_output=True, text=True, check=True).stdout
                for kernel in notes.split("- .agpr_count")[1:]:
                    out[re.search(r"\.name:\s+(\S+)", kernel)[1]] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel)[1])
            entry += 24 + length
        at = lib.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf not found")
def test_attention_kernels_keep_their_registers(tmp_path):
    found = {n: c for n, c in _spilled(tmp_path).items() if re.search(r"attn_(fwd|bwd)\w*_f16_kernel", n)}
    assert len(found) >= 15
    for name, count in found.items():
        assert count <= max((c for part, c in ALLOWED.items() if part in name), default=0), (name, count)

"""What the built scoring sweeps keep in registers: a spill inside their loops costs more than any schedule gains."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2506_08373_amd.binding import library_path

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(blob):
    """The gfx950 ELF images of the library's offload bundles (magic, entry count, then offset, size, id of each)."""
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.start() + 24
        (count,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(count):
            offset, size, id_len = struct.unpack_from("<QQQ", blob, at)
            if blob[at + 24:at + 24 + id_len].endswith(b"gfx950"):
                yield blob[m.start() + offset:m.start() + offset + size]
            at += 24 + id_len


def test_scoring_sweeps_do_not_spill(tmp_path):
    if not (os.path.exists(READELF) and os.path.exists(library_path())):
        pytest.skip("needs the built library and llvm-readelf")
    seen, spilled = 0, []
    with open(library_path(), "rb") as f:
        blob = f.read()
    for i, elf in enumerate(code_objects(blob)):
        path = tmp_path / ("%d.elf" % i)
        path.write_bytes(elf)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
            symbol = re.search(r"\.symbol:\s*(\S+)", kernel).group(1)
            if "score_kernel" not in symbol and "score_qs_kernel" not in symbol:
                continue
            seen += 1
            if int(re.search(r"\.vgpr_spill_count:\s*(\d+)", kernel).group(1)):
                spilled.append(symbol)
    assert seen > 100 and not spilled, spilled

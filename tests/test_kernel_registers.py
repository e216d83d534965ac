"""What the built scoring sweeps keep in registers: a spill inside their loops costs more than any schedule gains."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2506_08373_amd.binding import library_path

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"

PRUNED = ("prune_sample_rows_kernel", "prune_sweep_kernel", "prune_repair_kernel", "prune_sample_columns_kernel", "prune_listed_kernel")


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


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{symbol: (vector registers, spilled ones, bytes of private memory)} of the scoring kernels in the built library."""
    if not (os.path.exists(READELF) and os.path.exists(library_path())):
        pytest.skip("needs the built library and llvm-readelf")
    with open(library_path(), "rb") as f:
        blob = f.read()
    found = {}
    for i, elf in enumerate(code_objects(blob)):
        path = tmp_path_factory.mktemp("elf") / ("%d.elf" % i)
        path.write_bytes(elf)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
            symbol = re.search(r"\.symbol:\s*(\S+)", kernel).group(1)
            if any(name in symbol for name in ("score_kernel", "score_qs_kernel", *PRUNED)):
                found[symbol] = tuple(int(re.search(r"\." + key + r":\s*(\d+)", kernel).group(1))
                                      for key in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size"))
    # two 16-bit types, two head dimensions, one or two row blocks a wave; all but the sample's row statistics also by reduction
    assert [sum(name in symbol for symbol in found) for name in PRUNED] == [8, 16, 16, 16, 16]
    assert len(found) > 100
    return found


def test_scoring_sweeps_do_not_spill(kernels):
    assert not [symbol for symbol, (_, spilled, private) in kernels.items() if spilled or private]


@pytest.mark.parametrize("dtype", [0, 2])
@pytest.mark.parametrize("reduce_max", [0, 1])
def test_two_workgroups_of_the_eight_block_column_sweep_share_a_cu(kernels, dtype, reduce_max):
    """16-bit rows, d = 128, 8 waves x 1 row block: four waves per SIMD have 128 registers each."""
    name = "score_kernel_colsILi%dELi128ELi1ELi8ELi2ELi%dELb0EE" % (dtype, reduce_max)
    counts = [n for symbol, (n, *_) in kernels.items() if name in symbol]
    assert len(counts) == 1 and counts[0] <= 128

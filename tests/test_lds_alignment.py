"""Kernels access their dynamic LDS with 16-byte instructions, so it has to
start at a multiple of 16 bytes: behind the static LDS, which the compiler pads
to the alignment of the dynamic array's declaration."""
import glob
import os
import re
import subprocess

import pytest

from paper_2003_01178_amd import build

CSRC = build.CSRC


@pytest.mark.parametrize("src", sorted(os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "*.hip"))))
def test_dynamic_lds_arrays_are_declared_with_16_byte_alignment(src):
    with open(os.path.join(CSRC, src)) as f:
        for line in f:
            if "extern __shared__" in line:
                assert "__align__(16)" in line or " v4i " in line, line.strip()


def test_dynamic_lds_of_the_msb_shuffle_starts_at_16_bytes(tmp_path):
    """The kernel with both: its static LDS is the offset of its dynamic one."""
    if not os.path.exists(build.HIPCC):  # pragma: no cover - depends on the toolchain
        pytest.skip("no hipcc")
    asm = tmp_path / "msb_sort.s"
    subprocess.run([build.HIPCC, *build.CFLAGS, "-w", "--cuda-device-only", "-S", os.path.join(CSRC, "msb_sort.hip"),
                    "-o", str(asm)], check=True, capture_output=True)
    sizes, size = {}, None
    for line in asm.read_text().splitlines():   # a kernel's metadata gives its size before its name
        if m := re.match(r"\s*\.group_segment_fixed_size: (\d+)", line):
            size = int(m.group(1))
        elif (m := re.match(r"\s*\.name:\s+(_Z\S*)", line)) and "msb_shuffle" in m.group(1):
            sizes[m.group(1)] = size
    assert len(sizes) == 2
    for name, at in sizes.items():
        assert at % 16 == 0, name

"""The unstable radix shuffle's tile code (csrc/radix_tile.hpp), run on the CPU
with one fiber per lane: the LDS atomics of one instruction may serve the
lanes in any order, and no order may lose a pair of a partial tile."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


def test_unstable_shuffle_of_partial_tiles_in_any_lane_order(tmp_path):
    if not os.path.exists(CLANG):  # pragma: no cover - depends on the toolchain
        pytest.skip("no clang++")
    shutil.copy(os.path.join(ROOT, "paper_2003_01178_amd", "csrc", "radix_tile.hpp"), tmp_path)
    (tmp_path / "block.hpp").write_text("")     # the test defines what it uses of it
    exe = tmp_path / "lanes"
    subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-I", str(tmp_path), "-o", str(exe),
                    os.path.join(ROOT, "tests", "radix_tile_lanes.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]

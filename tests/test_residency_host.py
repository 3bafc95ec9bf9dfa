"""Registers and preloaded arguments of kernels whose launch rules count on how many workgroups share a compute unit, read from the
built code objects: 512 registers per SIMD lane, handed out in eights."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_18226_amd import build as B

BIN = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not os.path.exists(f"{BIN}/llvm-objdump"):
        pytest.skip("no llvm-objdump beside hipcc")
    if not os.path.exists(B.LIB_PATH):
        B.build_library()
    tmp = tmp_path_factory.mktemp("lib")
    subprocess.run([f"{BIN}/llvm-objdump", "--offloading", shutil.copy(B.LIB_PATH, tmp)], check=True, capture_output=True, cwd=tmp, timeout=60)
    return [str(tmp / n) for n in sorted(os.listdir(tmp)) if "gfx950" in n]


@pytest.fixture(scope="module")
def registers(code_objects):
    found = {}
    for path in code_objects:
        notes = subprocess.run([f"{BIN}/llvm-readelf", "--notes", path], check=True, capture_output=True, text=True, timeout=60).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            found[re.search(r"\.name:\s+(\S+)", kernel).group(1)] = int(re.search(r"\.vgpr_count:\s+(\d+)", kernel).group(1))
    return found


@pytest.mark.parametrize("kernel,waves", [       # mangled name and template arguments, waves per SIMD
    (r"k_selectILi256ELi1E", 7), (r"k_selectILi256ELi3ELi8E", 6), (r"k_selectILi512ELi(8|12|16)E", 4),
    (r"k_compact_planILi256ELi1E", 7), (r"k_compact_planILi(256|512)ELi2E", 6), (r"k_attend_gqaILi(64|128)ELi8E", 4),
    (r"k_compact_moveILi(4|8)E", 8), (r"k_compact_moveILi16E", 4), (r"k_compact_moveILi24E", 3), (r"k_compact_moveILi32E", 2),
])
def test_waves_per_simd(registers, kernel, waves):
    mine = {k: v for k, v in registers.items() if re.search(kernel, k)}
    assert mine
    for name, vgprs in mine.items():
        assert 512 // ((vgprs + 7) // 8 * 8) >= waves, (name, vgprs)


def test_row_moves_preload_eight_dwords(code_objects):
    """Most of their workgroups have nothing to move: what they cost is their launch, and each preloaded dword adds to it.  (A kernel
    with preloaded arguments begins with loads of just these, for firmware that does not preload.)"""
    seen = 0
    for path in code_objects:
        text = subprocess.run([f"{BIN}/llvm-objdump", "-d", "--no-show-raw-insn", "--mcpu=gfx950", path], check=True, capture_output=True,
                              text=True, timeout=60).stdout
        for kernel in re.findall(r"<\S*k_compact_moveILi\d+E\S*>:\n(.*?)s_branch", text, re.S):
            seen += 1
            assert sum(int(n or 1) for n in re.findall(r"s_load_dword(?:x(\d+))? ", kernel)) <= 8
    assert seen == 13                                        # (five tile sizes; four each with score rows, and with those and the records)

"""The attention kernels ask for entries of the slot list before they know how long it is, and rely on the bounds check of a buffer
load.  That check covers the vector offset and the instruction's own, not a scalar offset: the built code may not use one."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_18226_amd import build as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def test_buffer_loads_have_no_scalar_offset(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump beside hipcc")
    if not os.path.exists(B.LIB_PATH):
        B.build_library()
    lib = shutil.copy(B.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path, timeout=60)
    found, kernel = {}, None
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--mcpu=gfx950", name], check=True, capture_output=True, text=True,
                              cwd=tmp_path, timeout=60).stdout
        for line in text.splitlines():
            label = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            kernel = label.group(1) if label else kernel
            ins = re.match(r"\s*(buffer_\w+)\s+(.*?)\s*(//.*)?$", line)
            if ins and ins.group(1) not in ("buffer_wbl2", "buffer_inv"):
                # vdata, vaddr, srsrc, soffset and modifiers
                soffset = ins.group(2).split(", ")[3].split()[0]
                found.setdefault(kernel, []).append(soffset)
    assert sum("k_attend" in k for k in found) >= 16           # (the loads are there: every form of the two kernels has some)
    wrong = {k: sorted(set(v)) for k, v in found.items() if set(v) != {"0"}}
    assert not wrong, wrong

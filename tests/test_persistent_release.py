"""The compiled persistent kernel waits, in every wave that stores spikes past
its block's exchange line to the list buffer, for those stores before the
barrier after which another wave publishes their count (a barrier by itself
waits for no store)."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from paper_2109_12855_amd import sdeliver

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


def _kernels(tmp_path):
    so = shutil.copy(sdeliver.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(so)], check=True, capture_output=True,
                   cwd=tmp_path)
    out = {}
    for f in sorted(tmp_path.glob("lib.so.*gfx950*")):
        text = subprocess.run([OBJDUMP, "-d", str(f)], check=True, capture_output=True,
                              text=True).stdout
        for m in re.finditer(r"^[0-9a-f]+ <(\S*k_persist\S*)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text,
                             re.M | re.S):
            out[m[1]] = [re.sub(r"\s*//.*", "", x).strip() for x in m[2].splitlines()]
    return out


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_list_entries_are_out_before_the_barrier(tmp_path):
    kernels = _kernels(tmp_path)
    assert len(kernels) == 4, list(kernels)
    for name, code in kernels.items():
        agent = [i for i, x in enumerate(code)
                 if x.startswith("global_store_") and re.search(r"\bsc1\b", x)]
        line = max(i for i in agent if code[i].startswith("global_store_dwordx2"))
        entry = max(i for i in agent if code[i].startswith("global_store_dword ") and i < line)
        barrier = next(i for i in range(entry, line) if code[i] == "s_barrier")
        assert any(re.match(r"s_waitcnt\b.*vmcnt\(0\)", x) for x in code[entry:barrier]), (
            name, code[entry:barrier + 1])

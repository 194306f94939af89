"""A buffer store of 12 or 16 bytes whose offset comes from a scalar register was seen to store a vector register that the next
instruction had already overwritten, and the compiler puts no wait state between the two (it does where the scalar offset is
a constant): the built library has no such store."""
import os
import re
import subprocess

import pytest

from paper_2602_01410_amd import snip
from test_wait_states import OBJDUMP, code_objects


def with_scalar_offset(lines):
    """Stores like `buffer_store_dwordx4 v[2:5], v10, s[24:27], s65 offen`."""
    return [line for line in lines if re.search(r"buffer_store_dwordx[34]\s+\S+\s+\S+\s+s\[\d+:\d+\],\s+s\d+\b", line)]


def test_scan_finds_a_store_with_a_scalar_offset():
    bad = ["\tbuffer_store_dwordx4 v[2:5], v10, s[24:27], s65 offen // x", "\tbuffer_store_dwordx3 v[2:4], v10, s[24:27], s3 offen offset:16",
           "\tbuffer_store_dwordx4 v[2:5], off, s[24:27], s65"]
    good = ["\tbuffer_store_dwordx4 v[2:5], v10, s[24:27], 0 offen", "\tbuffer_store_dwordx2 v[2:3], v10, s[24:27], s65 offen",
            "\tbuffer_store_dwordx4 v[2:5], off, s[24:27], 0 offset:16", "\tglobal_store_dwordx4 v[0:1], v[2:5], off"]
    assert with_scalar_offset([line for pair in zip(bad + [""], good) for line in pair]) == bad


def test_library(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    stores = 0
    for i, obj in enumerate(code_objects(snip.LIB_PATH)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        out = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True, timeout=300).stdout.splitlines()
        stores += sum("buffer_store_dwordx4" in line for line in out)
        assert with_scalar_offset(out) == []
    assert stores > 0

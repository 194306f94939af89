"""A scalar register written by a vector instruction (v_readlane, v_readfirstlane, a compare) may be read by a memory
instruction five wait states later at the earliest.  The compiler keeps that distance for its own loads and not for those in
inline assembly, and it restores spilled scalar registers with v_readlane right in front of them; this looks at every memory
instruction of the built library."""
import os
import re
import struct
import subprocess

import pytest

from paper_2602_01410_amd import snip

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 5


def code_objects(path):
    with open(path, "rb") as f:
        blob = f.read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        base = m.start()
        n, = struct.unpack_from("<Q", blob, base + 24)
        p = base + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + idlen] and size:
                yield blob[base + off:base + off + size]
            p += 24 + idlen


def scalar(tok):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", tok)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", tok)
    return {int(m[1])} if m else {"vcc"} if tok.startswith("vcc") else set()


def too_close(lines):
    """(function, memory instruction, vector instruction, wait states between) of every pair below the distance."""
    found, seq, function, memory = [], [], "", 0
    for line in lines:
        if line.endswith(">:\n"):
            function, seq = line, []
            continue
        ins = line.split("//")[0].split()
        if not ins or not re.match(r"[a-z]+_", ins[0]):
            continue
        op, toks = ins[0], [t.rstrip(",") for t in ins[1:]]
        writes = set()
        if re.match(r"(global|buffer|flat|scratch)_", op):
            memory += 1
            reads = set().union(*[scalar(t) for t in toks])
            waited = 0
            for text, wr, states in reversed(seq):
                if waited >= WAIT_STATES:
                    break
                if wr & reads:
                    found.append((function.strip(), line.split("//")[0].strip(), text, waited))
                    break
                waited += states
        elif op.startswith("v_") and toks:
            writes = scalar(toks[0])
            if len(toks) > 1 and re.search(r"_co_|addc|subb|div_scale|mad_[ui]64", op):
                writes |= scalar(toks[1])
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            seq = []
        else:
            seq = (seq + [(" ".join(ins), writes, 1 + int(toks[0], 0) if op == "s_nop" else 1)])[-WAIT_STATES:]
    return found, memory


def test_scan_finds_a_pair_that_is_too_close():
    ins = ["0000 <k>:\n", " v_readlane_b32 s13, v255, 19 // x\n", " s_mov_b32 m0, s1\n", " s_nop 0\n", " global_load_lds_dword v1, s[12:13] // y\n"]
    assert [w for *_, w in too_close(ins)[0]] == [2]
    ins[3] = " s_nop 3\n"
    assert too_close(ins) == ([], 1)


def test_library(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    found, memory = [], 0
    for i, obj in enumerate(code_objects(snip.LIB_PATH)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        out = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True, timeout=300).stdout
        f, m = too_close(out.splitlines(keepends=True))
        found += f
        memory += m
    assert memory > 1000
    assert not found, (len(found), found[:5])

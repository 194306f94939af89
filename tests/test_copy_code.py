"""What the compiler makes of the GEMM kernels' copies, looked up in the built library.

A global->LDS copy waits until earlier ones have read the offsets that a vector instruction is about to write, so the stage loop
of the small GEMM tiles has to skip the cut of a last stage with a branch: no loop selects offsets between its barrier and the copies
that use them (64 x 32, [123 x 2240 x 17024] FP8: 28.9 us with selects, 23.0 with a branch).

The large tiles issue their copies between MFMAs, which hold a vector instruction up for about 20 cycles: hardly any spilled scalar
register is fetched back (v_readlane) there (256 x 128, [407 x 14080 x 14976] FP4 with fp32 results: 67.5 us with up to 39 of them in
a kernel, 62.5 with up to 16), and lane registers are not spilled to make room (256 x 256, [4960 x 1760 x 512] FP4 with bf16 results:
11.8 us with four of them and seven loads from scratch, 10.9 with one).

Results are stored streaming ("nt") or plain, by kernels of their own or by two branches of one, of which the compiler makes one plain store
if they differ in nothing else ([4096 x 2048 x 2048] FP4 16.0 us instead of 13.7).  So the stores are counted: as many of either kind as
a wave's part of the tile takes, twice that where whole tiles have stores without tests of their own ([4096 x 2048 x 2048] FP4, fp32
results on rows off 64 bytes, plain: 21.6 us on the stores of ragged tiles, 19.5 on those of whole ones)."""
import os
import re
import subprocess

import pytest

from paper_2602_01410_amd import snip
from test_wait_states import OBJDUMP, code_objects


def selects_before_copies(lines):
    """Copies whose offset register a v_cndmask wrote since the last barrier, with no branch between; and the number of copies."""
    found, copies, function, written = [], 0, "", None
    for line in lines:
        if line.endswith(">:"):
            function, written = line, None
            continue
        ins = line.split("//")[0].replace(",", " ").split()
        if not ins or "gemm_small_kernel" not in function:
            continue
        if ins[0] == "s_barrier":
            written = set()
        elif ins[0].startswith(("s_cbranch", "s_branch", "s_endpgm")):
            written = None
        elif written is not None and ins[0].startswith("v_cndmask"):
            written.add(ins[1])
        elif re.match(r"buffer_load_dword", ins[0]) and "lds" in ins:
            copies += 1
            if written is not None and ins[1] in written:
                found.append((function.strip(), line.split("//")[0].strip()))
    return found, copies


def test_scan_finds_a_select():
    loop = ["0000 <_Z17gemm_small_kernelv>:", " s_barrier", " v_cndmask_b32_e64 v2, v2, v3, s[4:5] // x", " buffer_load_dwordx4 v2, s[16:19], s4 offen lds"]
    assert len(selects_before_copies(loop)[0]) == 1
    loop.insert(2, " s_cbranch_scc1 4")
    assert selects_before_copies(loop) == ([], 1)


def fetched_between_mfmas(lines):
    """Kernel of the large tiles -> v_readlanes between s_setprio 1 and 0, the MFMA phases."""
    counts, function, inside = {}, "", False
    for line in lines:
        if line.endswith(">:"):
            function, inside = line, False
            if "gemm_fast_kernel" in line:
                counts[function] = 0
            continue
        ins = line.split("//")[0].split()
        if ins and function in counts:
            if ins[0] == "s_setprio":
                inside = ins[1] == "1"
            counts[function] += inside and ins[0] == "v_readlane_b32"
    return counts


def test_scan_counts_between_mfmas():
    body = ["0000 <_Z16gemm_fast_kernelv>:", " v_readlane_b32 s1, v2, 3", " s_setprio 1", " v_readlane_b32 s1, v2, 3 // x", " s_setprio 0", " v_readlane_b32 s1, v2, 3"]
    assert list(fetched_between_mfmas(body).values()) == [1]


def loads_from_scratch(lines):
    """Kernel of the large tiles -> scratch loads."""
    counts, function = {}, ""
    for line in lines:
        if line.endswith(">:"):
            function = line
        ins = line.split("//")[0].split()
        if ins and "gemm_fast_kernel" in function:
            counts[function] = counts.get(function, 0) + ins[0].startswith("scratch_load")
    return counts


def test_scan_counts_scratch_loads():
    body = ["0000 <_Z16gemm_fast_kernelv>:", " scratch_load_dword v0, off, off offset:12", " scratch_store_dword off, v0, off", "0100 <_Z1kv>:", " scratch_load_dword v0, off, off"]
    assert list(loads_from_scratch(body).values()) == [1]


def result_stores(lines):
    """GEMM kernel that takes grouped scales or the paper's -> 16-byte stores, streaming and plain."""
    counts, function = {}, ""
    for line in lines:
        if line.endswith(">:"):
            function = line
        ins = line.split("//")[0].split()
        if ins and re.search(r"gemm_(fast|small|paper|paper_wide)_kernel", function) and ins[0] == "global_store_dwordx4":
            kinds = counts.setdefault(function, [0, 0])
            kinds[0 if "nt" in ins else 1] += 1
    return counts


def wanted_stores(function):
    """What result_stores has to find in a kernel, by its mangled name: either of the pairs returned."""
    kernel, args = re.search(r"(gemm_(?:fast|small|paper_wide|paper)_kernel)(.*)", function).groups()
    f32 = re.match(r"ILi\dELi\dELb(\d)E", args).group(1) == "1"
    tile = re.search(r"Tile\w*?ILi\d+ELi\d+ELi(\d+)ELi(\d+)E", args)         # rows and columns of a workgroup, of a wave (the paper's recipe: 64 x 64)
    rows, columns = map(int, tile.groups()) if tile else (64, 64)
    n = rows * columns * (4 if f32 else 2) // 1024                              # a wave stores 1 KB at a time
    if kernel == "gemm_fast_kernel":
        return [2 * n, 0], [0, 2 * n]
    return ([2 * n, 2 * n],) if kernel == "gemm_paper_wide_kernel" else ([n, n],)


FAST = "0000 <_ZN4snip12_GLOBAL__N_116gemm_fast_kernelILi0ELi0ELb%dENS0_7TileCfgILi256ELi128ELi64ELi64ELi3ELi1EEELb0ELb1EEEvPKh>:"
SMALL = "0000 <_ZN4snip12_GLOBAL__N_117gemm_small_kernelILi0ELi0ELb0ENS0_9SmallTileILi32ELi32ELi32ELi32ELi8ELi4ELi2EEELb0EEEvPKh>:"


@pytest.mark.parametrize("function, streaming, plain, good", [
    (FAST % 0, 16, 0, True), (FAST % 0, 0, 16, True), (FAST % 1, 32, 0, True), (FAST % 1, 0, 32, True), (SMALL, 2, 2, True),
    (FAST % 0, 8, 8, False),            # streaming for ragged tiles only
    (FAST % 1, 0, 16, False),           # no stores without tests for whole tiles
    (SMALL, 0, 2, False)])              # one plain store of two branches
def test_scan_counts_result_stores(function, streaming, plain, good):
    body = [function] + [" global_store_dwordx4 v0, v[2:5], s[0:1] nt // x"] * streaming + [" global_store_dwordx4 v0, v[2:5], s[0:1] // nt"] * plain
    found = result_stores(body + ["0100 <_Z1kv>:", " global_store_dwordx4 v0, v[2:5], s[0:1]"])
    assert list(found.values()) == [[streaming, plain]]
    assert (found[function] in wanted_stores(function)) == good


def test_library(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    copies, fetched, scratch, stores = 0, {}, {}, {}
    for i, obj in enumerate(code_objects(snip.LIB_PATH)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        out = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True, timeout=300).stdout.splitlines()
        found, n = selects_before_copies(out)
        assert found == []
        copies += n
        fetched.update(fetched_between_mfmas(out))
        scratch.update(loads_from_scratch(out))
        stores.update(result_stores(out))
    assert copies > 100
    assert len(fetched) > 10 and max(fetched.values()) <= 20
    assert scratch.keys() == fetched.keys() and max(scratch.values()) <= 3
    assert len(stores) > 60 and {f: n for f, n in stores.items() if n not in wanted_stores(f)} == {}
    fast = [n for f, n in stores.items() if "gemm_fast_kernel" in f]
    assert sum(n[0] > 0 for n in fast) == sum(n[1] > 0 for n in fast) == len(fast) // 2

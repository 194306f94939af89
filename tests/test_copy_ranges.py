"""The source ranges of the GEMM kernels' copies through buffer descriptors (csrc/copy_ranges.h), compiled for the host: over
row counts, contraction extents and stages, those past the last included, the uniform offset never exceeds the size, what is in
range lies inside the operand and belongs to the stage, and what does not exist is out of range."""
import os
import subprocess

import paper_2602_01410_amd

CSRC = os.path.join(os.path.dirname(paper_2602_01410_amd.__file__), "csrc")

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include "copy_ranges.h"
using namespace snip;

#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s (rows %d, extent %d, stage %d)\n", __LINE__, #c, rows, r, st); std::exit(1); } } while (0)
static bool in_range(CopyRange c, unsigned lane) { return lane < c.size - c.uniform; }      // unsigned, as the hardware may do it

int main()
{
    long checks = 0;
    const int kRows[] = {1, 31, 129, 256, 300, 1000}, kExtents[] = {32, 96, 128, 160, 256, 288, 384, 416, 640, 1184, 4128};
    for (int rows : kRows) for (int r : kExtents) for (int fp4 = 0; fp4 < 2; ++fp4) for (int ng = 1; ng < 3; ++ng) for (int tile = 32; tile <= 256; tile *= 2) {
        const int ke = 128 * ng, nstage = (r + ke - 1) / ke, ngrp = (r + 127) / 128;
        const unsigned row_bytes = fp4 ? r / 2 : r, step = fp4 ? ke / 2 : ke, pitch = (rows + 255) / 256 * 256 * 4;
        for (int i0 = 0; i0 < rows; i0 += tile) for (int st = 0; st < nstage + 9; ++st, ++checks) {
            const unsigned bytes = (rows - i0 < tile ? rows - i0 : tile) * row_bytes;
            const CopyRange c = code_range(st, nstage, bytes, step);
            CHECK(c.uniform <= c.size);
            for (int row = 0; row < tile; row += 5) for (unsigned b = 0; b < step; b += 16) {
                if (st == nstage - 1 && b >= row_bytes - st * step) break;             // such lanes have no source
                const unsigned lane = row * row_bytes + b;
                CHECK(in_range(c, lane) == (st < nstage && i0 + row < rows));
                CHECK(!in_range(c, lane) || lane + c.uniform + 16 <= bytes);
            }
            const CopyRange s = scale_range(st, nstage, ngrp, ng, pitch, i0 * 4);
            CHECK(s.uniform <= s.size);
            // a wave's second copy of a stage (64 rows on, tiles of 128 and 256 rows) in the uniform offset: there up to the last stage
            if (tile >= 128 && st < nstage) {
                const CopyRange t{s.size, s.uniform + 256};
                CHECK(t.uniform <= t.size);
                for (int g = 0; g < ng; ++g) for (int row = 0; row < tile - 64; ++row)
                    CHECK(in_range(t, scale_lane(g, row, pitch)) == (st * ng + g < ngrp));
            }
            for (int g = 0; g < ng; ++g) for (int row = 0; row < tile; ++row) {
                const unsigned lane = scale_lane(g, row, pitch);
                CHECK(in_range(s, lane) == (st * ng + g < ngrp && st < nstage));
                CHECK(!in_range(s, lane) || i0 * 4 + s.uniform + lane == (unsigned)(st * ng + g) * pitch + (i0 + row) * 4);
            }
            CHECK(!in_range(c, 0x80000000u) && !in_range(s, 0x80000000u));
        }
    }
    // the largest grouped scale copies: nothing wraps in 32 bits
    for (long long pitch = 1024; pitch <= 1ll << 30; pitch *= 4) {
        const int ngrp = (int)(((1ll << 31) - 1) / pitch), rows = (int)(pitch / 4), r = ngrp * 128;
        for (int ng = 1; ng < 3; ++ng) for (int st = 0, n = (ngrp + ng - 1) / ng; st < n; st += st < n - 2 && n > 1000 ? n / 1000 : 1) {
            const unsigned row0 = (unsigned)pitch - 1024;
            CHECK(descriptor_covers(ngrp * pitch) && !descriptor_covers((ngrp + 1) * pitch));
            const CopyRange s = scale_range(st, n, ngrp, ng, (unsigned)pitch, row0);
            CHECK(s.size == ngrp * pitch - row0 && s.uniform == (long long)st * ng * pitch && s.uniform <= s.size);
            for (int g = 0; g < ng; ++g) CHECK(in_range(s, scale_lane(g, 255, (unsigned)pitch)) == (st * ng + g < ngrp));
        }
    }
    std::printf("%ld\n", checks);
}
"""


def run(tmp_path, program, include=CSRC):
    src = tmp_path / "ranges.cpp"
    src.write_text(program)
    exe = tmp_path / "ranges"
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{include}", str(src), "-o", str(exe)], check=True, timeout=120)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)


def test_ranges(tmp_path):
    res = run(tmp_path, PROGRAM)
    assert res.returncode == 0, res.stdout
    assert int(res.stdout) > 10000


# what the kernels did before: the size 0 past the last stage beside an offset that kept growing
def test_offset_past_the_size_is_noticed(tmp_path):
    with open(os.path.join(CSRC, "copy_ranges.h")) as f:
        text = f.read()
    wrong = text.replace("CopyRange{0u, 0u}", "CopyRange{0u, (unsigned)st}")
    assert wrong != text
    (tmp_path / "copy_ranges.h").write_text(wrong)
    res = run(tmp_path, PROGRAM, tmp_path)
    assert res.returncode == 1 and "c.uniform <= c.size" in res.stdout

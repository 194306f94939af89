"""The rules by which launchers choose between kernels (csrc/picks.h), compiled for the host, against what both sides take on an
MI355X."""
import os
import subprocess

import paper_2602_01410_amd

CSRC = os.path.join(os.path.dirname(paper_2602_01410_amd.__file__), "csrc")

# GEMMs of the paper's recipe that the two kernels differ on by 10 % or more: I, J, R, FP4 x FP4, B in tiles, scales on 16 bytes: us with 128 x 128, with 256 x 128 (256 compute units)
MEASURED = [
    # a little more than whole rounds of 256 x 128, long contractions whose scales are copied one by one
    (4992, 1792, 7040, 0, 0, 0, 97.1, 122.0), (4992, 1792, 7040, 0, 1, 0, 114.3, 151.5), (4992, 1792, 7040, 1, 0, 0, 73.6, 90.9),
    (4992, 1792, 7040, 1, 1, 0, 90.1, 122.7), (6911, 1368, 7040, 0, 0, 0, 100.7, 122.2), (2816, 6784, 6272, 1, 1, 0, 131.9, 166.0),
    (4252, 6272, 8064, 0, 1, 0, 300.0, 354.6), (3200, 7640, 3840, 1, 0, 0, 86.0, 95.4), (2048, 5120, 7168, 1, 1, 1, 88.8, 102.2),
    (3072, 3072, 7168, 0, 1, 1, 116.9, 134.7),
    # whole rounds
    (4096, 8192, 2048, 0, 0, 1, 98.5, 81.9), (4096, 8192, 2048, 1, 0, 1, 65.8, 52.9), (4096, 2048, 8192, 0, 0, 1, 89.0, 73.9),
    (4096, 2048, 8192, 0, 1, 1, 100.0, 89.0), (4096, 2048, 8192, 1, 0, 1, 58.3, 47.6), (4096, 2048, 8192, 1, 1, 1, 74.0, 66.0),
    (8192, 2048, 4096, 0, 1, 1, 103.0, 93.0), (8192, 2048, 4096, 1, 1, 1, 78.0, 68.7), (8192, 8192, 8192, 0, 1, 1, 790.0, 685.0),
    (5120, 2560, 4608, 1, 1, 1, 79.7, 68.9),
]

# GEMMs of the 32 x 32 tile: operands cached, stages: us with one stage per barrier, with two
STAGES = [(1, 1, 3.26, 3.38), (1, 3, 3.52, 3.60), (1, 16, 5.40, 4.95), (1, 32, 7.24, 6.76), (0, 62, 37.2, 38.5)]

# one-pass quantize: rows, columns, bytes of a stored column, statistics: us with turns of eight units, with an eighth per XCD
ORDERS = [(1504, 2080, 752, 0, 5.9, 5.8), (2432, 4896, 1216, 1, 21.8, 21.6), (32768, 4096, 16384, 0, 87.9, 103.0), (8160, 8160, 8160, 0, 82.3, 89.6),
          (2048, 22016, 1024, 0, 35.8, 38.8), (6144, 22016, 6144, 0, 118.4, 124.5), (8192, 32768, 4096, 0, 199.9, 186.2), (8192, 28672, 8192, 0, 206.3, 198.5),
          (4096, 4096, 2048, 1, 23.7, 27.7), (10496, 23808, 10496, 0, 226.9, 211.6), (12544, 21504, 12544, 0, 224.4, 210.3), (4224, 30080, 4224, 0, 107.2, 113.6)]

# ... in turns: columns, bytes of a stored column: us with pairs of row units, with four
BANDS = [(2048, 43040, 154.8, 129.0), (2048, 26000, 96.7, 81.1), (6144, 14304, 159.4, 137.0), (11008, 4080, 90.4, 84.2), (1984, 12880, 49.2, 43.7),
         (8160, 4080, 54.3, 60.9), (11008, 8192, 127.6, 130.7), (4096, 16384, 87.2, 89.6), (8288, 11312, 160.6, 174.1)]

# ... columns, units: us with tiles read directly, through LDS
LDS = [(32, 1100, 9.24, 10.23), (64, 537, 7.08, 7.79), (96, 537, 8.87, 8.84), (11008, 11008, 140.5, 126.9), (4096, 8192, 101.2, 87.7), (2048, 256, 5.9, 6.3),
       (3072, 576, 12.5, 11.4), (4096, 800, 14.4, 15.2)]

# ... forms for large tensors: rows, columns, FP8 rows, FP8 columns, statistics, us with codes stored plainly, streamed: of the quantize call ([12384 x
# 10656]), of a step of one linear, of a block ([16384 x 11008] FP4, [8192 x 28672], [32768 x 8192])
STREAMED = [(16384, 11008, 0, 0, 0, 4638., 4675.), (8192, 28672, 0, 0, 0, 8966., 9021.), (32768, 8192, 0, 0, 0, 3606., 3572.),
            (16384, 4096, 0, 0, 0, 184.4, 192.5), (16384, 4096, 0, 1, 0, 246.6, 262.0), (16384, 4096, 1, 0, 0, 249.9, 252.0), (16384, 4096, 1, 1, 0, 294.0, 278.3),
            (4096, 16384, 1, 1, 0, 301.4, 284.9), (16384, 11008, 1, 0, 0, 1050., 1013.), (16384, 11008, 0, 1, 0, 1041., 1021.),
            (16384, 4096, 1, 1, 1, 318.9, 308.6), (4096, 16384, 1, 1, 1, 336.0, 313.4), (4096, 16384, 0, 1, 1, 302.4, 289.6), (8192, 8192, 1, 0, 1, 434.6, 425.0),
            (2176, 8960, 0, 0, 0, 102.4, 117.0), (12384, 10656, 0, 0, 0, 160.8, 196.3), (12384, 10656, 0, 0, 1, 160.8, 196.3)]

# GEMMs of the small tiles: one row of tiles, bytes of B's codes, us with B read plainly, streamed: forwards of three blocks in turn, one GEMM on
# weights in turn (90 MB and 541 MB; 268 MB)
B_STREAMED = [(1, 11008 * 2048, 62.9, 56.4), (1, 9536 * 1792, 47.8, 56.9), (0, 11008 * 2048, 9.24, 12.46), (0, 11008 * 2048, 11.25, 13.10), (0, 16384 * 4096, 19.54, 25.88)]

# GEMM results: address, pitch in elements, fp32, us stored plainly, streamed
RESULTS = [(0, 2080, 0, 15.1, 13.1), (0, 5200, 0, 27.9, 32.5), (0, 2064, 1, 17.99, 16.92), (16, 2064, 1, 21.79, 29.02), (32, 3088, 1, 73.07, 94.35),
           (16, 4128, 0, 39.89, 42.70), (32, 1056, 0, 4.23, 4.63), (16, 1056, 0, 4.23, 4.64)]

# ... direct: units, us with columns stored by all waves, by those of columns
APART = [(8, 3.70, 3.45), (204, 5.80, 5.48), (256, 6.53, 6.33), (512, 10.81, 11.39), (704, 11.40, 12.16)]


def run(tmp_path, expression, args):
    src, exe = tmp_path / "pick.cpp", tmp_path / "pick"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "picks.h"\nint main(int n, char** v) { auto a = [&](int i) { return std::atoll(v[i + 1]); };\n'
                   f'std::printf("%d", (int)({expression})); }}\n')
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True, timeout=120)
    return [int(subprocess.run([str(exe), *map(str, row)], capture_output=True, text=True, check=True, timeout=60).stdout) for row in args]


def test_paper_kernel(tmp_path):
    picks = run(tmp_path, "snip::paper_wide_pays(a(0), a(1), a(2), a(3), a(4), a(5), 256)", [m[:6] for m in MEASURED])
    assert picks == [int(m[7] < m[6]) for m in MEASURED]


def test_stages_per_barrier(tmp_path):
    assert run(tmp_path, "snip::small_stages_per_barrier(a(0), a(1))", [m[:2] for m in STAGES]) == [2 if m[3] < m[2] else 1 for m in STAGES]


def test_unit_order(tmp_path):
    picks = run(tmp_path, "snip::qb_eighths(a(0), a(1), a(1), a(2), a(3))", [m[:4] for m in ORDERS])
    assert picks == [int(m[5] < m[4]) for m in ORDERS]


def test_bands(tmp_path):
    picks = run(tmp_path, "snip::qb_band_log2(a(0), a(1))", [m[:2] for m in BANDS])
    assert picks == [1 + int(m[3] < m[2]) for m in BANDS]


def test_through_lds(tmp_path):
    picks = run(tmp_path, "snip::qb_through_lds(a(0), a(1), 256)", [m[:2] for m in LDS])
    assert picks == [int(m[3] < m[2]) for m in LDS]


def test_streamed_codes(tmp_path):
    rule = "snip::qb_streams(a(0), a(1), a(2), a(3), a(4), a(5), a(6))"
    assert run(tmp_path, rule, [(*m[:5], 0, 0) for m in STREAMED]) == [int(m[6] < m[5]) for m in STREAMED]
    # codes that start off 64 bytes have rows off 64 bytes, whatever their pitch
    for stats in (0, 1):
        assert run(tmp_path, rule, [(16384, 11008, 1, 1, stats, *at) for at in ((4096, 64), (16, 0), (0, 48), (32, 32))]) == [1, 0, 0, 0]


def test_streamed_weights(tmp_path):
    picks = run(tmp_path, "snip::small_streams_b(a(0), a(1))", [m[:2] for m in B_STREAMED])
    assert picks == [int(m[3] < m[2]) for m in B_STREAMED]


def test_streamed_results(tmp_path):
    picks = run(tmp_path, "snip::streams_result(a(0), a(1), a(2))", [m[:3] for m in RESULTS])
    assert picks == [int(m[4] < m[3]) for m in RESULTS]


def test_rows_apart(tmp_path):
    picks = run(tmp_path, "snip::qb_rows_apart(a(0), 256)", [m[:1] for m in APART])
    assert picks == [int(m[2] < m[1]) for m in APART]


ORDER_PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "picks.h"
using namespace snip;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s (row units %d, whole %d, column groups %d, eighth %d)\n", __LINE__, #c, nru, whole, ncg, eighth); return 1; } } while (0)
int main()
{
    for (int nru = 1; nru <= 21; ++nru) for (int whole = nru - 1; whole <= nru; ++whole) for (int ncg = 1; ncg <= 40; ++ncg) for (int in_turns = 0; in_turns < 2; ++in_turns) for (int log2 = 1; log2 <= 1 + in_turns; ++log2) {
        const int units = nru * ncg, eighth = in_turns ? 0 : (units + 7) / 8, end = eighth ? 8 * eighth : (units + 63) / 64 * 64;
        const int bands = qb_bands(whole, nru, eighth, log2), band = 1 << log2;
        std::vector<int> seen(units, 0);
        for (int v = 0; v < end; ++v) {
            const int u = qb_unit(v, eighth);
            if (u >= units) continue;
            const QbPlace p = qb_place(u, bands, log2, ncg);
            CHECK(u >= 0 && p.ru >= 0 && p.ru < nru && p.cg >= 0 && p.cg < ncg);
            ++seen[p.ru * ncg + p.cg];
            // short units come last, of all or, in eighths, of their pair
            if (in_turns) CHECK((u >= whole * ncg) == (p.ru >= whole));
            // an XCD's eight in a row are two row units by four column groups, or four by two
            if (in_turns && u % 8 == 0 && u + 7 < bands * band * ncg && u % (band * ncg) + 7 < band * ncg && u % (band * ncg) % band == 0) {
                const QbPlace q = qb_place(u + 7, bands, log2, ncg);
                CHECK(p.ru % band == 0 && q.ru == p.ru + band - 1 && q.cg == p.cg + 8 / band - 1 && qb_unit(v + 56, eighth) == u + 7);
            }
        }
        CHECK(std::all_of(seen.begin(), seen.end(), [](int n) { return n == 1; }));
    }
    return 0;
}
"""


def test_every_unit_once_and_short_ones_last(tmp_path):
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(ORDER_PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{CSRC}", str(src), "-o", str(exe)], check=True, timeout=120)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout

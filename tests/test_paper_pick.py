"""The rule that gives a GEMM of the paper's recipe to the 128 x 128 or the 256 x 128 kernel (csrc/paper_pick.h), compiled for the
host: on problems where the two differ by 10 % or more on an MI355X it takes the faster one."""
import os
import subprocess

import paper_2602_01410_amd

CSRC = os.path.join(os.path.dirname(paper_2602_01410_amd.__file__), "csrc")

# I, J, R, FP4 x FP4, B in tiles, scales on 16 bytes: us with 128 x 128, with 256 x 128 (256 compute units)
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

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "paper_pick.h"
int main(int argc, char** argv)
{
    for (int i = 1; i + 5 < argc; i += 6)
        std::printf("%d\n", snip::paper_wide_pays(atoll(argv[i]), atoll(argv[i + 1]), atoll(argv[i + 2]), atoi(argv[i + 3]), atoi(argv[i + 4]), atoi(argv[i + 5]), 256));
}
"""


def test_the_faster_kernel(tmp_path):
    src, exe = tmp_path / "pick.cpp", tmp_path / "pick"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{CSRC}", str(src), "-o", str(exe)], check=True, timeout=120)
    picks = subprocess.run([str(exe)] + [str(v) for m in MEASURED for v in m[:6]], capture_output=True, text=True, check=True, timeout=120).stdout.split()
    assert len(picks) == len(MEASURED)
    for m, wide in zip(MEASURED, picks):
        assert (wide == "1") == (m[7] < m[6]), m

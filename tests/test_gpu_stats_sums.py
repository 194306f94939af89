"""Workgroup sums of the statistics passes keep what their waves' fp32 sums hold: a workgroup whose first wave has the sum
2^24 and whose others have 1 delivers 2^24 + 3, which fp32 cannot hold (its neighbours are 2^24 + 2 and 2^24 + 4)."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


# the four waves of a workgroup: tiles below each other (one unit) or side by side (a unit each)
@pytest.mark.parametrize("call,unit,shape", [("stats_both", None, (128, 128)), ("stats_both", None, (32, 512)),
                                             ("chosen", "4x4", (128, 128)), ("chosen", "wave", (32, 512)), ("both_formats", "4x4", (128, 128)),
                                             ("both_formats", "4x8", (128, 128)), ("both_formats", "wave", (32, 512))])
def test_workgroup_sums_are_not_rounded(call, unit, shape, monkeypatch):
    snip = require_gpu()
    if unit:
        monkeypatch.setenv("SNIP_QUANT_BOTH_UNIT", unit)
    x = torch.zeros(shape, device="cuda", dtype=torch.bfloat16)
    for k in range(4):
        x[(32 * k, 0) if shape[0] == 128 else (0, 128 * k)] = 4096.0 if k == 0 else 1.0
    for fmt in (snip.FP8, snip.FP4):
        row, col = snip.alloc_stats(), snip.alloc_stats()
        if call == "stats_both":
            snip.snip_quant_error_stats_both(x, out_row=row, out_col=col)
        else:
            snip.snip_quantize_both(x, fmt, fmt, stats_row=row, stats_col=col, both_formats=call == "both_formats")
        assert row[0].item() == col[0].item() == 2.0 ** 24 + 3
        field = 2 if fmt == snip.FP8 else 1
        assert row[field].item() == col[field].item() == 0.0


def test_column_sums_of_squares_are_exact_on_constant_columns():
    """65536 rows of one value per column, its square an odd number of 16 bits: 32 of them are 21 bits, and 32 such blocks of a
    lane 26 bits with five zeros at the end.  fp32 holds each of these sums (not each of 1024 squares added one by one), and
    the lanes' sums are added in double."""
    snip = require_gpu()
    rows, cols = 65536, 160
    values = (torch.arange(cols, device="cuda") % 64 * 2 + 129).double() / 128
    x = values.bfloat16().expand(rows, cols).contiguous()
    lines = torch.empty((cols, 3), dtype=torch.float32, device="cuda")
    total = snip.snip_quant_error_stats(x, snip.COL, per_line=lines)
    want = rows * values.square()
    assert torch.equal(lines[:, 0].double(), want)
    # a wave adds 64 lanes' sums of two columns in fp32: seven roundings
    assert abs(float(total[0]) / float(want.sum()) - 1) <= 7 * 2.0 ** -24

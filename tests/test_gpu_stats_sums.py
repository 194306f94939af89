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

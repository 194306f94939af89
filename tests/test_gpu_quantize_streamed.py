"""snip_quantize_both of tensors large enough for their codes to be streamed (64 M elements, stored rows on 64 bytes) and just not
(stored rows off 64 bytes), without statistics and with: the bytes of the two single-orientation calls."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stats", [False, True])
@pytest.mark.parametrize("shape", [(8192, 8192), (8320, 8256), (8224, 8224)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
def test_bytes(shape, fmts, stats):
    snip = require_gpu()
    rows, cols = shape
    assert rows * cols >= 64 << 20
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn((rows, cols), generator=gen, device="cuda").bfloat16()
    x[:, ::97] *= 50.0
    qr, qc = snip.alloc_qtensor(rows, cols, fmts[0]), snip.alloc_qtensor(cols, rows, fmts[1])
    for q in (qr, qc):
        q.codes.fill_(0xA5)
        q.scales.fill_(0xA5)
    rec = torch.zeros(6, dtype=torch.float64, device="cuda") if stats else None
    snip.snip_quantize_both(x, *fmts, snip.NO_OVERFLOW, out_row=qr, out_col=qc, both_formats=stats,
                            **({"stats_row": rec[:3], "stats_col": rec[3:]} if stats else {}))
    for axis, got in ((snip.ROW, qr), (snip.COL, qc)):
        want = snip.snip_quantize(x, got.fmt, axis)
        assert torch.equal(got.codes, want.codes) and torch.equal(got.scales, want.scales)
    if stats:
        # sums in fp32 per lane and wave, double across them (bound of test_gpu_stats.py)
        assert float(rec[0]) == pytest.approx(float(x.double().square().sum()), rel=1e-5) and float(rec[3]) == pytest.approx(float(rec[0]), rel=1e-5)

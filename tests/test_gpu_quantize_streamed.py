"""snip_quantize_both of tensors large enough for their codes to be streamed (128 MB in both orientations, 256 MB in FP4 alone, with
statistics 64 M elements, stored rows on 64 bytes) and just not (smaller, or stored rows off 64 bytes by their pitch or by where the
codes start), without statistics and with: the bytes of the two single-orientation calls."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stats", [False, True])
@pytest.mark.parametrize("shape", [(8192, 8192), (8320, 8256), (8224, 8224)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
def test_bytes(shape, fmts, stats):
    check(shape, fmts, stats)


# every pair of formats streamed, and with codes that start off 64 bytes
@pytest.mark.parametrize("stats", [False, True])
@pytest.mark.parametrize("shape, fmts, start", [((8192, 11264), (0, 1), 0), ((8320, 11264), (1, 0), 0), ((16384, 16448), (1, 1), 0), ((8192, 8192), (0, 0), 48)])
def test_bytes_by_formats(shape, fmts, start, stats):
    check(shape, fmts, stats, start)


def check(shape, fmts, stats, start=0):
    snip = require_gpu()
    rows, cols = shape
    assert rows * cols >= 64 << 20
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn((rows, cols), generator=gen, device="cuda").bfloat16()
    x[:, ::97] *= 50.0
    qr, qc = snip.alloc_qtensor(rows, cols, fmts[0]), snip.alloc_qtensor(cols, rows, fmts[1])
    for q in (qr, qc):
        q.codes = torch.empty(start + q.codes.numel(), dtype=torch.uint8, device="cuda")[start:].view(q.codes.shape)
        assert q.codes.data_ptr() % 64 == start
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

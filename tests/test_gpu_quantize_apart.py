"""snip_quantize_both read directly, with the columns stored by the waves of columns alone (up to a unit per compute unit) and by all
(more): row units of one to four tiles (waves without a tile meet the same barriers), ragged columns, rows that hold no whole number of
dwords of scales: the bytes of the two single-orientation calls."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(32, 32), (64, 416), (96, 128), (160, 1248), (2048, 2048), (4128, 1312), (4192, 1056)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
def test_bytes(shape, fmts, monkeypatch):
    snip = require_gpu()
    rows, cols = shape
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = (torch.randn((rows, cols), generator=gen, device="cuda") * 10.0 ** (4 * torch.rand((rows, 1), generator=gen, device="cuda") - 2)).bfloat16()
    monkeypatch.setenv("SNIP_QUANT_BOTH_UNIT", "4x4")
    qr, qc = snip.alloc_qtensor(rows, cols, fmts[0]), snip.alloc_qtensor(cols, rows, fmts[1])
    for q in (qr, qc):
        q.codes.fill_(0xA5)
        q.scales.fill_(0xA5)
    snip.snip_quantize_both(x, *fmts, snip.NO_OVERFLOW, out_row=qr, out_col=qc)
    for axis, got in ((snip.ROW, qr), (snip.COL, qc)):
        want = snip.snip_quantize(x, got.fmt, axis)
        assert torch.equal(got.codes, want.codes) and torch.equal(got.scales, want.scales)

"""snip_quantize_both with tiles that go through LDS (no statistics), where that can go wrong: row units of one to four tiles, a
last column group of 32, 64 and 96 columns, sources inside wider ones, more units than a turn of eight per XCD: the bytes of the
two single-orientation calls, and of the direct form."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(32, 32), (64, 160), (96, 96), (128, 128), (160, 1248), (1056, 2112)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("rule", [0, 1])
def test_bytes(shape, fmts, rule, monkeypatch):
    snip = require_gpu()
    rows, cols = shape
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    buf = torch.randn((rows, cols + 40), generator=gen, device="cuda") * 10.0 ** (4 * torch.rand((rows, 1), generator=gen, device="cuda") - 2)
    x = buf.bfloat16()[:, 8:8 + cols]
    runs = []
    for form in ("4x4", "lds"):
        monkeypatch.setenv("SNIP_QUANT_BOTH_UNIT", form)
        qr, qc = snip.alloc_qtensor(rows, cols, fmts[0]), snip.alloc_qtensor(cols, rows, fmts[1])
        for q in (qr, qc):
            q.codes.fill_(0xA5)
            q.scales.fill_(0xA5)
            q.scales_g4.fill_(0xA5)
        snip.snip_quantize_both(x, *fmts, rule, out_row=qr, out_col=qc)
        runs.append([t for q in (qr, qc) for t in (q.codes, q.scales, q.scales_g4)])
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    for axis, fmt, got in ((snip.ROW, fmts[0], runs[1][:2]), (snip.COL, fmts[1], runs[1][3:5])):
        want = snip.snip_quantize(x, fmt, axis, rule)
        assert torch.equal(got[0], want.codes) and torch.equal(got[1], want.scales)

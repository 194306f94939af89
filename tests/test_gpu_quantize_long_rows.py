"""snip_quantize_both on rows so far apart that the offsets inside a tile do not fit 32 bits: the bytes of the two
single-orientation calls, sums of the statistics pass (1e-5: fp32 sums per lane in another order)."""
import numpy as np
import pytest
import torch

from gpu_util import host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stats", [0, 1, 2])
@pytest.mark.parametrize("ld", [(1 << 25) - 8, 1 << 25])         # the last that fits and the first that does not
def test_row_stride(ld, stats):
    snip = require_gpu()
    rows, cols = 64, 160
    src = torch.randn((rows, cols), generator=torch.Generator(device="cuda").manual_seed(ld + stats), device="cuda").bfloat16()
    buf = torch.empty((rows - 1) * ld + cols, dtype=torch.bfloat16, device="cuda")
    x = buf.as_strided((rows, cols), (ld, 1))
    x.copy_(src)
    st = torch.zeros(6, dtype=torch.float64, device="cuda")
    kw = dict(stats_row=st[:3], stats_col=st[3:], workspace=snip.alloc_workspace(rows, cols), both_formats=stats == 2) if stats else {}
    qr, qc = snip.snip_quantize_both(x, snip.FP4, snip.FP8, 0, **kw)
    for axis, fmt, got in ((snip.ROW, snip.FP4, qr), (snip.COL, snip.FP8, qc)):
        want = snip.snip_quantize(src, fmt, axis, 0)
        assert torch.equal(got.codes, want.codes) and torch.equal(got.scales, want.scales)
        if stats:
            ref, s = host(snip.snip_quant_error_stats(src, axis, 0)), host(st)[3 * axis:3 * axis + 3]
            fields = [0, 1, 2] if stats == 2 else [0, 1 if fmt == snip.FP4 else 2]
            assert stats == 2 or np.isnan(s[3 - fields[1]])
            np.testing.assert_allclose(s[fields], ref[fields], rtol=1e-5)

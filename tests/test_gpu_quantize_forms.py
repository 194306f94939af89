"""snip_quantize_both in each of its work distributions, at unit counts where they can go wrong (an odd number of row
units, a last unit with fewer tiles, ragged columns, fewer units than XCDs): the bytes of the two single-orientation calls,
and the sums of the statistics pass (1e-5: fp32 sums per lane in another order, as everywhere)."""
import numpy as np
import pytest
import torch

from gpu_util import host, require_gpu

pytestmark = pytest.mark.gpu


def check(rows, cols, fr, fc, rule, stats, pad=8):
    snip = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(rows * 31 + cols)
    x = torch.randn((rows, cols + pad), generator=gen, device="cuda", dtype=torch.float32).bfloat16()[:, :cols]
    qr, qc = snip.alloc_qtensor(rows, cols, fr), snip.alloc_qtensor(cols, rows, fc)
    for q in (qr, qc):
        q.codes.fill_(0xA5)
        q.scales.fill_(0xA5)
    st = torch.zeros(6, dtype=torch.float64, device="cuda")
    ws = snip.alloc_workspace(rows, cols)
    kw = dict(stats_row=st[:3], stats_col=st[3:], workspace=ws, both_formats=stats == 2) if stats else {}
    snip.snip_quantize_both(x, fr, fc, rule, out_row=qr, out_col=qc, **kw)
    for axis, fmt, got in ((snip.ROW, fr, qr), (snip.COL, fc, qc)):
        want = snip.snip_quantize(x, fmt, axis, rule)
        assert torch.equal(got.codes, want.codes) and torch.equal(got.scales, want.scales)
        # (the grouped copy: rows of the tensor, blocks that exist)
        sr, nblk = want.scales.shape
        for q in (got, want):
            assert q.scales_g4 is not None
        g = [q.scales_g4.view(-1, (sr + 255) // 256 * 256, 4)[:, :sr].permute(1, 0, 2).reshape(sr, -1)[:, :nblk] for q in (got, want)]
        assert torch.equal(*g)
        if stats:
            ref = host(snip.snip_quant_error_stats(x, axis, rule))
            s = host(st)[:3] if axis == snip.ROW else host(st)[3:]
            if stats == 1:
                other = 2 if fmt == snip.FP4 else 1
                assert np.isnan(s[other])
                s[other] = ref[other]
            np.testing.assert_allclose(s, ref, rtol=1e-5)


@pytest.mark.parametrize("shape", [(32, 32), (160, 96), (416, 1056), (1120, 352)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("stats", [0, 1, 2])
def test_small(shape, fmts, stats, quant_both_unit):
    check(*shape, *fmts, 0, stats)


# the library's own choice: four waves with two tiles each (12 M ... 48 M elements, FP4 columns; 48 M = 50331648: just below and
# just above), a wave per unit (beyond, FP8 columns from 28 M); without statistics tiles through LDS, with rows of more than 16384
# columns in either order of the units; with the written formats' statistics a wave per unit from 56 M on, where it fills its
# rounds, or four waves with two tiles each
@pytest.mark.parametrize("shape,fmts,stats", [((3232, 4128), (1, 1), 2), ((3232, 4128), (0, 1), 2), ((8224, 6112), (1, 1), 2), ((8224, 6176), (1, 1), 2),
                                              ((8224, 4128), (0, 0), 2), ((8224, 6176), (1, 0), 0), ((16672, 8096), (1, 1), 0),
                                              ((16672, 8096), (0, 1), 0), ((16672, 8096), (0, 0), 0), ((16672, 8096), (1, 1), 1), ((4096, 16512), (0, 0), 0), ((2080, 16512), (1, 1), 0),
                                              ((8192, 7392), (1, 1), 1), ((8192, 7392), (0, 0), 1), ((8224, 8224), (0, 1), 1), ((3232, 6624), (0, 1), 1)])
def test_large(shape, fmts, stats):
    check(*shape, *fmts, 1 if stats == 0 else 0, stats, 128 if shape[1] > 16384 else 8)

"""The small GEMM tiles of one or two waves, of which 32 x 32 takes two pipeline stages per barrier: every number of stages around
their rings, whole last stages and cut ones, bit for bit against the general kernel (which the oracle checks)."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", ["32x32", "64x32"])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1)])
def test_numbers_of_stages(fmts, tile, monkeypatch):
    snip = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(11)
    plan = snip.make_plan((*fmts, 0, 0, 0, 0))
    ke = 256 if fmts == (1, 1) else 128
    for stages in range(1, 20):
        for R in (stages * ke - 32, stages * ke):
            q = []
            for rows, fmt in ((70, fmts[0]), (97, fmts[1])):
                q.append(snip.snip_quantize(torch.randn((rows, R), generator=gen, device="cuda").bfloat16(), fmt, snip.ROW))
                if R // 32 % 4:                         # bytes the layout leaves unspecified: worst case, "not a number"
                    q[-1].scales_g4[-1, :, R // 32 % 4:] = 0xFF
            outs = []
            for t in ("general", tile):
                monkeypatch.setenv("SNIP_GEMM_TILE", t)
                outs.append(snip.snip_gemm_fwd(plan, *q, out=torch.empty((70, 104), dtype=torch.float32, device="cuda")[:, :97], out_dtype=1).clone())
            assert torch.equal(*outs), (stages, R)


@pytest.mark.parametrize("tile", ["32x32", "64x32"])
def test_large_operands(tile, monkeypatch):
    """Operands of more than 10 MB take one stage per barrier."""
    snip = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(12)
    plan = snip.make_plan((0, 1, 0, 0, 0, 0))
    a, b = (torch.randn((r, 2208), generator=gen, device="cuda").bfloat16() for r in (70, 9800))
    q = snip.snip_quantize(a, 0, snip.ROW), snip.snip_quantize(b, 1, snip.ROW)
    assert q[0].codes.numel() + q[1].codes.numel() > 10e6
    outs = []
    for t in ("general", tile):
        monkeypatch.setenv("SNIP_GEMM_TILE", t)
        outs.append(snip.snip_gemm_fwd(plan, *q, out_dtype=1).clone())
    assert torch.equal(*outs)

"""The 256 x 128 GEMM tile (three stage buffers and one phase a stage, two and two for contractions of two stages) against the
256 x 256 one (two and two) and the general kernel: all add the products of an output element in the same order, so every byte
of the result agrees.  Stage counts: the fewest of either, and up to two more (each start of the ring of buffers for a second
tile), whole and cut last stages; one tile, tiles that end a row and a few columns after another, ragged tiles, more tiles than
compute units (the next tile's first stages are copied before the result is stored)."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("stages", [2, 3, 4, 5])
@pytest.mark.parametrize("cut", [0, 96])
@pytest.mark.parametrize("shape", [(256, 256), (257, 136), (300, 200), (4400, 2300)])
def test_same_bytes_in_both_tiles(shape, cut, stages, fmts, monkeypatch):
    snip = require_gpu()
    i, j = shape
    r = stages * (256 if fmts == (1, 1) else 128) - cut
    assert i > 128 and j > 128                                   # with two stages and more: what the two large tiles take
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    a = snip.snip_quantize(torch.randn((i, r), generator=gen, device="cuda").bfloat16(), fmts[0], snip.ROW)
    b = snip.snip_quantize(torch.randn((j, r), generator=gen, device="cuda").bfloat16(), fmts[1], snip.ROW)
    plan = snip.make_plan((fmts[0], fmts[1]) * 3)
    ld = (j + 7) // 8 * 8
    for dtype, tdtype in ((snip.OUT_BF16, torch.bfloat16), (snip.OUT_FP32, torch.float32)):
        got = []
        for tile in ("big", "wide", "general"):
            monkeypatch.setenv("SNIP_GEMM_TILE", tile)
            out = torch.zeros((i, ld), dtype=tdtype, device="cuda")
            snip.snip_gemm_fwd(plan, a, b, out=out[:, :j], out_dtype=dtype)
            got.append(out)
        assert bool(got[0].any())
        assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])

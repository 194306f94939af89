"""Few tokens through a weight of 20 MB and more, whose codes the small GEMM tiles stream: one row of tiles, weights that end inside a
tile, contractions that end inside a stage: the general kernel's bytes."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", [(1, 11008, 4096), (33, 10410, 4128), (64, 4100, 11040)])
def test_same_bytes(shape, fmts, monkeypatch):
    snip = require_gpu()
    i, j, r = shape
    assert j * r // 2 >= 20 << 20
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    a, b = (snip.snip_quantize(torch.randn((n, r), generator=gen, device="cuda").bfloat16(), f, snip.ROW) for n, f in ((i, fmts[0]), (j, fmts[1])))
    plan = snip.make_plan(fmts * 3)
    ld = (j + 7) // 8 * 8
    for dtype, tdtype in ((snip.OUT_BF16, torch.bfloat16), (snip.OUT_FP32, torch.float32)):
        got = []
        for tile in ("64x64", "64x32", "32x32", "general"):
            monkeypatch.setenv("SNIP_GEMM_TILE", tile)
            out = torch.full((i, ld), 7.0, dtype=tdtype, device="cuda")
            snip.snip_gemm_fwd(plan, a, b, out=out[:, :j], out_dtype=dtype)
            got.append(out)
        assert bool((got[0][:, j:] == 7.0).all())
        assert all(torch.equal(got[-1], g) for g in got)

"""Tile of 32 x 64, which stands for 64 x 64 up to 32 rows: the general kernel's bytes, and nothing outside the result; 33 rows for the
other side.  Outputs that end inside a tile, contractions of one stage, of less and more than the ring of six, and cut ones."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", [(1, 33, 32), (31, 64, 256), (32, 65, 1312), (32, 200, 1536), (17, 8224, 3360), (33, 130, 1824)])
def test_same_bytes(shape, fmts, monkeypatch):
    snip = require_gpu()
    i, j, r = shape
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    a, b = (snip.snip_quantize(torch.randn((n, r), generator=gen, device="cuda").bfloat16(), f, snip.ROW) for n, f in ((i, fmts[0]), (j, fmts[1])))
    plan = snip.make_plan(fmts * 3)
    for dtype, tdtype in ((snip.OUT_BF16, torch.bfloat16), (snip.OUT_FP32, torch.float32)):
        for ld in ((j + 7) // 8 * 8, (j + 31) // 32 * 32):               # plain and streaming stores
            got = []
            for tile in ("64x64", "general"):
                monkeypatch.setenv("SNIP_GEMM_TILE", tile)
                out = torch.full((i + 2, ld), 7.0, dtype=tdtype, device="cuda")
                snip.snip_gemm_fwd(plan, a, b, out=out[:i, :j], out_dtype=dtype)
                got.append(out)
            assert bool((got[0][i:] == 7.0).all()) and bool((got[0][:, j:] == 7.0).all())
            assert torch.equal(got[0], got[1])

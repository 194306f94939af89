"""The 256 x 128 GEMM tile against the 256 x 256 one and the general kernel, with output norms: every byte of the result agrees
(all add the products of an output element in the same order), and each tile's norm is that of its result.  Shapes: two and
three stages, extents that end inside a tile, a stage or a scale group, more tiles than compute units."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", [(256, 256, 512), (129, 300, 544), (513, 130, 1056), (1000, 1160, 4128), (4400, 2200, 768), (2048, 4096, 2048)])
def test_same_bytes_and_norm(shape, fmts, monkeypatch):
    snip = require_gpu()
    i, j, r = shape
    assert i > 128 and j > 128 and r > (256 if fmts == (1, 1) else 128)      # what the two large tiles take (a tile that cannot serve is not used)
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    a = snip.snip_quantize(torch.randn((i, r), generator=gen, device="cuda").bfloat16(), fmts[0], snip.ROW)
    b = snip.snip_quantize(torch.randn((j, r), generator=gen, device="cuda").bfloat16(), fmts[1], snip.ROW)
    plan = snip.make_plan((fmts[0], fmts[1]) * 3)
    ld = (j + 7) // 8 * 8
    for dtype, tdtype in ((snip.OUT_BF16, torch.bfloat16), (snip.OUT_FP32, torch.float32)):
        got = {}
        for tile in ("wide", "big", "general"):
            monkeypatch.setenv("SNIP_GEMM_TILE", tile)
            out = torch.zeros((i, ld), dtype=tdtype, device="cuda")
            norm = torch.zeros(1, dtype=torch.float64, device="cuda")
            ws = torch.empty(snip.gemm_workspace_bytes(i, j), dtype=torch.uint8, device="cuda")
            snip.snip_gemm_fwd_norm(plan, a, b, out=out[:, :j], out_dtype=dtype, sum_sq=norm, workspace=ws)
            got[tile] = out
            # fp32 sums of squares per lane, wave and workgroup (bound of test_gpu_gemm.py)
            assert float(norm[0]) == pytest.approx(float(out.double().square().sum()), rel=5e-6), tile
        assert bool(got["wide"].any())
        assert torch.equal(got["wide"], got["big"]) and torch.equal(got["wide"], got["general"])

"""GPU parity of the GEMM tiles that serve small and ragged outputs, and of contraction extents that end inside a
pipeline stage: every tile against the oracle and, bit for bit, against the general kernel (all of them add an
element's products in the same order)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_01410_amd import workloads as wl

from gpu_util import host, rel_fro, require_gpu, to_dev

pytestmark = pytest.mark.gpu
TILES = ("32x32", "64x32", "64x64", "128x128", "wide", "big")
TOL_F32 = 1e-4       # the bound of test_gpu_gemm.py for fp32 outputs

# rows, columns, contraction: one row; edges of a 32 x 32 tile; edges of 64 / 128 tiles with a contraction of one block, of
# one block more than a stage, with and without a second scale group in the last FP4 stage; the ring wrapping several times
SHAPES = [(1, 72, 32), (31, 40, 96), (33, 96, 160), (65, 136, 288), (129, 200, 416), (257, 264, 1184), (64, 520, 2336)]


def operands(snip, rng, shape, fa, fb):
    I, J, R = shape
    a = wl.f32_to_bf16_bits((rng.standard_normal((I, R)) * 2.0 ** rng.integers(-4, 4, size=(I, 1))).astype(np.float32))
    b = wl.f32_to_bf16_bits(rng.standard_normal((J, R)).astype(np.float32))
    qs = [snip.snip_quantize(to_dev(t), f, snip.ROW) for t, f in ((a, fa), (b, fb))]
    for q in qs:                                   # bytes the layout leaves unspecified: worst case, "not a number"
        nb = R // 32
        if nb % 4:
            q.scales_g4[-1, :, nb % 4:] = 0xFF
        q.scales_g4[:, q.rows:, :] = 0xFF
    want = oracle.gemm_fwd(oracle.fake_quant(a, fa, oracle.ROW), oracle.fake_quant(b, fb, oracle.ROW))
    return qs, want


@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_tile_matches_oracle_and_general_kernel(shape, fa, fb, monkeypatch):
    snip = require_gpu()
    I, J, R = shape
    (aq, bq), want = operands(snip, np.random.default_rng(9100 + I + fa * 2 + fb), shape, fa, fb)
    plan = snip.make_plan((fa, fb, 0, 0, 0, 0))
    outs = {}
    for tile in ("general",) + TILES:
        monkeypatch.setenv("SNIP_GEMM_TILE", tile)
        for dt, name in ((torch.float32, "f32"), (torch.bfloat16, "bf16")):
            buf = torch.full((I + 1, J + 16), 7.0, dtype=dt, device="cuda")      # a margin that must stay as it is
            snip.snip_gemm_fwd(plan, aq, bq, out=buf[:I, :J], out_dtype=1 if dt == torch.float32 else 0)
            torch.cuda.synchronize()
            assert torch.all(buf[I:] == 7.0) and torch.all(buf[:, J:] == 7.0), tile
            outs[tile, name] = host(buf[:I, :J].float())
    assert rel_fro(outs["general", "f32"].astype(np.float64), want) <= TOL_F32
    for (tile, name), got in outs.items():
        assert np.array_equal(got, outs["general", name]), (tile, name)


@pytest.mark.parametrize("fmt", [0, 1])
def test_norm_with_ragged_contraction(fmt, monkeypatch):
    """Output norms: the tiles that deliver one partial per workgroup, with a last stage that is not whole."""
    snip = require_gpu()
    (aq, bq), _ = operands(snip, np.random.default_rng(9200 + fmt), (300, 392, 864), fmt, fmt)
    plan = snip.make_plan((fmt,) * 6)
    for tile in ("128x128", "wide", "big", "32x32", "none"):
        monkeypatch.setenv("SNIP_GEMM_TILE", tile)
        y, nrm = snip.snip_gemm_fwd_norm(plan, aq, bq, out_dtype=1)
        torch.cuda.synchronize()
        # fp32 sums of squares per lane, wave and workgroup (bound of test_gpu_gemm.py)
        assert float(nrm[0]) == pytest.approx(float(y.double().square().sum()), rel=5e-6), tile


@pytest.mark.parametrize("tile", TILES)
def test_no_scale_behind_the_last_group_is_read(tile, monkeypatch):
    """FP4 with an odd number of scale groups, several tiles each way: the last stage's second group does not exist.  Behind
    the grouped copies lie bytes that mean "not a number"."""
    snip = require_gpu()
    i, j, r = 520, 648, 1152
    gen = torch.Generator(device="cuda").manual_seed(7)
    qs = []
    for rows in (i, j):
        q = snip.alloc_qtensor(rows, r, snip.FP4)
        n = q.scales_g4.numel()
        q.scales_g4 = torch.full((n + 64 * 1024,), 0xFF, dtype=torch.uint8, device="cuda")[:n].view(q.scales_g4.shape)
        snip.snip_quantize(torch.randn((rows, r), generator=gen, device="cuda").bfloat16(), snip.FP4, snip.ROW, out=q)
        qs.append(q)
    outs = []
    for t in ("general", tile):
        monkeypatch.setenv("SNIP_GEMM_TILE", t)
        outs.append(snip.snip_gemm_fwd((snip.FP4,) * 6, *qs, out_dtype=snip.OUT_FP32))
    assert bool(torch.isfinite(outs[0]).all()) and torch.equal(*outs)

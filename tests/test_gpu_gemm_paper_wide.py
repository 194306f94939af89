"""GPU parity of the 256 x 128 tile of snip_gemm_paper where it changes what it does: three stages (the least it takes) and
more, odd numbers of slabs, chunks of scales that do not fill a fetch or do not start on 16 bytes, ragged tiles, more tiles than
compute units.  Products, factors and their order are those of the 128 x 128 tile, so the bits have to be the same; both are checked
against the oracle too (test_gpu_gemm_paper.py)."""
import pytest
import torch

import oracle
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

T, B = oracle.TILE_1x128, oracle.BLOCK_128x128


def both_tiles(snip, monkeypatch, qa, qb, I, J, dtype):
    ld, tdtype = (J + 7) // 8 * 8 + 8, torch.float32 if dtype == snip.OUT_FP32 else torch.bfloat16
    runs = []
    for tile in ("128x128", "256x128"):
        monkeypatch.setenv("SNIP_GEMM_PAPER_TILE", tile)
        buf = torch.full((I, ld), 7.0, dtype=tdtype, device="cuda")
        snip.snip_gemm_paper(*qa, *qb, out=buf[:, :J], out_dtype=dtype)
        runs.append(buf)
    assert bool((runs[1][:, J:] == 7.0).all())
    return runs[0][:, :J], runs[1][:, :J]


def operand(snip, gen, rows, cols, fmt, group):
    # rows and slabs of very different size, so that a factor taken from the wrong row or slab shows
    x = torch.randn((rows, cols), generator=gen, device="cuda") * 10.0 ** (4 * torch.rand((rows, 1), generator=gen, device="cuda") - 2)
    x *= (10.0 ** (2 * torch.rand((1, cols // 128), generator=gen, device="cuda") - 1)).repeat_interleave(128, 1)
    return (*snip.snip_quantize_paper(x.bfloat16(), fmt, snip.ROW, group), fmt, group)


@pytest.mark.parametrize("groups", [(T, T), (T, B), (B, T), (B, B)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", [(1, 1, 640), (256, 128, 768), (257, 391, 640), (300, 200, 1024), (600, 130, 1152), (515, 260, 1664), (4352, 2200, 896)])
def test_same_bits_as_the_small_tile(shape, fmts, groups, monkeypatch):
    snip = require_gpu()
    I, J, R = shape
    gen = torch.Generator(device="cuda").manual_seed(I * 31 + J * 7 + R)
    qa, qb = operand(snip, gen, I, R, fmts[0], groups[0]), operand(snip, gen, J, R, fmts[1], groups[1])
    for dtype in (snip.OUT_FP32, snip.OUT_BF16):
        small, wide = both_tiles(snip, monkeypatch, qa, qb, I, J, dtype)
        assert torch.equal(small, wide)


# Three stages and four (FP8 and mixed formats; FP4 x FP4 has three in 640 above): a tile of less than one fetch of scales and of
# exactly one, alone and with a second tile per workgroup
@pytest.mark.parametrize("groups", [(T, T), (T, B)])
@pytest.mark.parametrize("fmts", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", [(300, 200, 384), (300, 200, 512), (4352, 2200, 384), (4352, 2200, 512)])
def test_short_contractions(shape, fmts, groups, monkeypatch):
    snip = require_gpu()
    I, J, R = shape
    gen = torch.Generator(device="cuda").manual_seed(I + J + R)
    qa, qb = operand(snip, gen, I, R, fmts[0], groups[0]), operand(snip, gen, J, R, fmts[1], groups[1])
    small, wide = both_tiles(snip, monkeypatch, qa, qb, I, J, snip.OUT_FP32)
    assert torch.equal(small, wide)


@pytest.mark.parametrize("groups", [(T, T), (T, B)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1)])
def test_scales_off_16_bytes(fmts, groups, monkeypatch):
    snip = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(3)
    I, J, R = 300, 260, 1024
    qa, qb = operand(snip, gen, I, R, fmts[0], groups[0]), operand(snip, gen, J, R, fmts[1], groups[1])
    moved = torch.empty(qa[1].numel() + 1, dtype=torch.float32, device="cuda")[1:].view(qa[1].shape)
    moved.copy_(qa[1])
    assert moved.data_ptr() % 16 == 4
    small, wide = both_tiles(snip, monkeypatch, (qa[0], moved, *qa[2:]), qb, I, J, snip.OUT_FP32)
    assert torch.equal(small, wide)


@pytest.mark.parametrize("group_a", [T, B])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
def test_non_finite_group_stays_in_its_column(fmts, group_a, monkeypatch):
    # more tiles than compute units: a workgroup's second tile must not see the factors or products of its first one
    snip = require_gpu()
    monkeypatch.setenv("SNIP_GEMM_PAPER_TILE", "256x128")
    I, J, R = 17 * 256, 17 * 128, 640
    if 17 * 17 <= torch.cuda.get_device_properties(0).multi_processor_count:
        pytest.fail("the shape needs more tiles")
    gen = torch.Generator(device="cuda").manual_seed(5)
    a, b = torch.randn((I, R), generator=gen, device="cuda").bfloat16(), torch.randn((J, R), generator=gen, device="cuda").bfloat16()
    qa = (*snip.snip_quantize_paper(a, fmts[0], snip.ROW, group_a), fmts[0], group_a)
    bad = torch.tensor([t * 128 + 64 * (t % 2) + 32 + t for t in range(17)], device="cuda")
    runs = []
    for poison in (False, True):
        if poison:
            b[bad, R - 1] = float("inf")
        qb = (*snip.snip_quantize_paper(b, fmts[1], snip.ROW, T), fmts[1], T)
        runs.append(snip.snip_gemm_paper(*qa, *qb, out_dtype=snip.OUT_FP32))
    clean, got = runs
    others = torch.ones(J, dtype=torch.bool, device="cuda")
    others[bad] = False
    assert bool(torch.isnan(got[:, bad]).all())
    assert torch.equal(got[:, others], clean[:, others])

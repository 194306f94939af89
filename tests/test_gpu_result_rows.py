"""Results whose rows start on 64 bytes (streaming stores) and 16 bytes past that (plain ones, by their pitch or by where the result starts),
in every GEMM kernel that makes the difference: whole tiles and ragged ones, the same bytes in both, the general kernel's too, and nothing written between the rows."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

TILES = ("big", "wide", "128x128", "64x64", "64x32", "32x32", "general")


def result(run, i, j, pad, tdtype, start=0):
    buf = torch.full((i, j + pad), 7.0, dtype=tdtype, device="cuda")
    run(buf[:, start:start + j])
    assert bool((buf[:, :start] == 7.0).all()) and bool((buf[:, start + j:] == 7.0).all())
    return buf[:, start:start + j]


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("shape", [(256, 256, 768), (512, 1216, 768), (300, 264, 800)])
def test_rows_on_and_off_64_bytes(shape, f32, monkeypatch):
    snip = require_gpu()
    i, j, r = shape
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    a, b = (snip.snip_quantize(torch.randn((n, r), generator=gen, device="cuda").bfloat16(), snip.FP4, snip.ROW) for n in (i, j))
    plan, dtype, tdtype = snip.make_plan((snip.FP4,) * 6), int(f32), torch.float32 if f32 else torch.bfloat16
    got = []
    for tile in TILES:
        monkeypatch.setenv("SNIP_GEMM_TILE", tile)
        for pad in (-j % 32, -j % 32 + 16 // (4 if f32 else 2)):
            got.append(result(lambda out: snip.snip_gemm_fwd(plan, a, b, out=out, out_dtype=dtype), i, j, pad, tdtype))
    assert bool(got[0].any())
    assert all(torch.equal(got[0], g) for g in got[1:])


@pytest.mark.parametrize("shape", [(256, 256, 768), (1032, 1024, 512), (300, 264, 896)])
def test_rows_on_and_off_64_bytes_paper(shape, monkeypatch):
    snip = require_gpu()
    i, j, r = shape                                        # (1032 x 1024: more elements than the 128 x 128 tile stores plainly in any case)
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    qa, qb = ((*snip.snip_quantize_paper(torch.randn((n, r), generator=gen, device="cuda").bfloat16(), snip.FP4, snip.ROW, g), snip.FP4, g)
              for n, g in ((i, snip.TILE_1x128), (j, snip.BLOCK_128x128)))
    got = []
    for tile in ("128x128", "256x128"):
        monkeypatch.setenv("SNIP_GEMM_PAPER_TILE", tile)
        for pad in (-j % 32, -j % 32 + 8):
            got.append(result(lambda out: snip.snip_gemm_paper(*qa, *qb, out=out), i, j, pad, torch.bfloat16))
    assert bool(got[0].any())
    assert all(torch.equal(got[0], g) for g in got[1:])


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("shape", [(256, 256, 768), (300, 264, 800)])
def test_start_off_64_bytes(shape, f32, monkeypatch):
    snip = require_gpu()
    i, j, r = shape
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    a, b = (snip.snip_quantize(torch.randn((n, r), generator=gen, device="cuda").bfloat16(), snip.FP8, snip.ROW) for n in (i, j))
    plan, dtype, tdtype, piece = snip.make_plan((snip.FP8,) * 6), int(f32), torch.float32 if f32 else torch.bfloat16, 16 // (4 if f32 else 2)
    got = []
    for tile in TILES:
        monkeypatch.setenv("SNIP_GEMM_TILE", tile)
        for start in (0, piece, 3 * piece):
            got.append(result(lambda out: snip.snip_gemm_fwd(plan, a, b, out=out, out_dtype=dtype), i, j, -j % 32 + 32, tdtype, start))
    assert bool(got[0].any())
    assert all(torch.equal(got[0], g) for g in got[1:])


def test_start_off_64_bytes_paper(monkeypatch):
    snip = require_gpu()
    i, j, r = 1032, 1024, 512
    gen = torch.Generator(device="cuda").manual_seed(i + j + r)
    qa, qb = ((*snip.snip_quantize_paper(torch.randn((n, r), generator=gen, device="cuda").bfloat16(), snip.FP8, snip.ROW, g), snip.FP8, g)
              for n, g in ((i, snip.TILE_1x128), (j, snip.BLOCK_128x128)))
    got = []
    for tile in ("128x128", "256x128"):
        monkeypatch.setenv("SNIP_GEMM_PAPER_TILE", tile)
        for start in (0, 8, 24):
            got.append(result(lambda out: snip.snip_gemm_paper(*qa, *qb, out=out), i, j, 32, torch.bfloat16, start))
    assert bool(got[0].any())
    assert all(torch.equal(got[0], g) for g in got[1:])

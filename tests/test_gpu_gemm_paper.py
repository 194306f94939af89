"""GPU parity of snip_gemm_paper where its kernels change what they do: odd and even numbers of 128-element slabs (FP4 x FP4
takes two per stage), fewer slabs than stage buffers, ragged tiles, more tiles than compute units, every pair of scaling
groups.  Both kernels (SNIP_GEMM_PAPER_TILE; 256 x 128 where it can serve the call) against the float64 product of the oracle's
dequantized operands."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2602_01410_amd import workloads as wl

from gpu_util import host, require_gpu, to_dev

pytestmark = pytest.mark.gpu

T, B = oracle.TILE_1x128, oracle.BLOCK_128x128


def operand(snip, rng, rows, cols, fmt, group):
    # rows and slabs of very different size, so that a factor taken from the wrong row or slab shows
    a = rng.standard_normal((rows, cols)) * 10.0 ** rng.uniform(-2, 2, size=(rows, 1))
    a *= np.repeat(10.0 ** rng.uniform(-1, 1, size=(1, cols // 128)), 128, axis=1)
    bits = wl.f32_to_bf16_bits(a.astype(np.float32))
    codes, scales = snip.snip_quantize_paper(to_dev(bits), fmt, snip.ROW, group)
    oc, os_ = oracle.quantize_paper(bits, fmt, oracle.ROW, group)
    return (codes, scales, fmt, group), np.asarray(oracle.dequantize_paper(oc, os_, fmt, group), dtype=np.float64)


@pytest.mark.parametrize("groups", [(T, T), (T, B), (B, T), (B, B)])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", [(1, 1, 128), (128, 128, 256), (130, 72, 384), (257, 391, 640), (96, 300, 1152), (2200, 2050, 384), (4352, 2200, 640)])
def test_gemm_paper(shape, fmts, groups, monkeypatch):
    snip = require_gpu()
    I, J, R = shape
    rng = np.random.default_rng([I, J, R, *fmts, *groups])
    (qa, a), (qb, b) = operand(snip, rng, I, R, fmts[0], groups[0]), operand(snip, rng, J, R, fmts[1], groups[1])
    want = a @ b.T
    # The matrix core adds the 64 products of an instruction with a shared alignment: bits more than 13 places below the
    # largest product are dropped (an element of four products, 44.2, 9.0, 4.0 and 0.06, came out off by 0.0054), so the
    # error of an element is bounded by 2^-12 of the sum of its products' magnitudes (measured over these inputs: up to
    # 1.04e-4 of it, the same bits from every kernel with this instruction) and by 2^-8 of itself once rounded to bf16.
    # A factor taken from a wrong row, column or slab is off by a multiple of the magnitudes.
    mags = np.abs(a) @ np.abs(b).T
    ld = (J + 7) // 8 * 8
    outs = ((snip.OUT_FP32, torch.float32, 0.0), (snip.OUT_BF16, torch.bfloat16, 2.0 ** -8))
    for tile, (dtype, tdtype, own) in itertools.product(("128x128", "256x128"), outs):
        monkeypatch.setenv("SNIP_GEMM_PAPER_TILE", tile)
        buf = torch.full((I, ld), 7.0, dtype=tdtype, device="cuda")
        snip.snip_gemm_paper(*qa, *qb, out=buf[:, :J], out_dtype=dtype)
        torch.cuda.synchronize()
        got = host(buf[:, :J].to(torch.float64))
        assert (np.abs(got - want) <= 2.0 ** -12 * mags + own * np.abs(want)).all()
        assert bool((buf[:, J:] == 7.0).all())


@pytest.mark.parametrize("group_a", [T, B])
@pytest.mark.parametrize("fmts", [(0, 0), (1, 1), (0, 1), (1, 0)])
def test_non_finite_group_stays_in_its_column(fmts, group_a, monkeypatch):
    # More tiles than compute units: a workgroup's second tile must not see the factors of its first one's last slab.  One
    # infinity per 128 rows of B, in the last slab, always at another offset (two tiles with the same one would hide it).
    snip = require_gpu()
    monkeypatch.setenv("SNIP_GEMM_PAPER_TILE", "128x128")
    n, R = 17 * 128, 256
    if (n // 128) ** 2 <= torch.cuda.get_device_properties(0).multi_processor_count:
        pytest.fail("the shape needs more tiles")
    gen = torch.Generator(device="cuda").manual_seed(5)
    a, b = (torch.randn((n, R), generator=gen, device="cuda").bfloat16() for _ in range(2))
    qa = (*snip.snip_quantize_paper(a, fmts[0], snip.ROW, group_a), fmts[0], group_a)
    bad = torch.tensor([t * 128 + 64 * (t % 2) + 32 + t for t in range(n // 128)], device="cuda")
    runs = []
    for poison in (False, True):
        if poison:
            b[bad, R - 1] = float("inf")
        qb = (*snip.snip_quantize_paper(b, fmts[1], snip.ROW, T), fmts[1], T)
        runs.append(snip.snip_gemm_paper(*qa, *qb, out_dtype=snip.OUT_FP32))
    clean, got = runs
    others = torch.ones(n, dtype=torch.bool, device="cuda")
    others[bad] = False
    assert bool(torch.isnan(got[:, bad]).all())
    assert torch.equal(got[:, others], clean[:, others])

"""The native half of the Python binding on the CPU: what is not a CUDA tensor, a QTensor or a plan is refused with a
Python exception, before anything reaches the library."""
import subprocess
import sys

import pytest
import torch

from paper_2602_01410_amd import snip


def test_wrong_arguments_raise():
    q = snip.alloc_qtensor(32, 64, snip.FP8, device="cpu")
    with pytest.raises(ValueError, match="2-D CUDA tensor"):
        snip.snip_quantize(torch.zeros((32, 64), dtype=torch.bfloat16), snip.FP8, out=q)
    with pytest.raises(TypeError):
        snip._nat().quantize([1, 2], 0, 0, 0, q, None, None, None)
    with pytest.raises(AttributeError):
        snip._nat().gemm(0, snip.make_plan((0,) * 6), object(), q, torch.zeros((32, 32)), 0, 0)
    with pytest.raises(TypeError, match="arguments"):
        snip._nat().gemm(0)
    with pytest.raises(ValueError, match="no such GEMM"):
        snip._nat().gemm(3, snip.make_plan((0,) * 6), q, q, torch.zeros((32, 32)), 0, 0)


def test_library_status_becomes_an_exception():
    q, other = (snip.alloc_qtensor(32, c, snip.FP8, device="cpu") for c in (64, 96))
    with pytest.raises(snip.SnipError) as e:                 # contraction extents differ: refused by the library on the host
        snip.snip_gemm_fwd((0,) * 6, q, other, out=torch.zeros((32, 32), dtype=torch.bfloat16), stream=0)
    assert e.value.status == 4
    with pytest.raises(snip.SnipError) as e:                 # operand format differs from the plan
        snip.snip_gemm_wgrad((0, 0, 0, 0, 1, 1), q, q, out=torch.zeros((32, 32), dtype=torch.bfloat16), stream=0)
    assert e.value.status == 3


def test_library_without_the_native_half():
    """Sizes, host functions and operands need the library alone: the native half is tied to one torch."""
    code = """
import sys
sys.modules["paper_2602_01410_amd._snip_binding"] = None          # importing it raises
from paper_2602_01410_amd import snip
assert snip.workspace_bytes(32, 64) > 0 and snip.alloc_qtensor(32, 64, snip.FP8, device="cpu").codes.shape == (32, 64)
assert snip.snip_loss_divergence(1.0, 1.0, 1, 1.0, 1.0, 1, 1) > 0
try:
    snip._nat()
except ImportError:
    print("refused")
"""
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.strip() == "refused", res.stderr

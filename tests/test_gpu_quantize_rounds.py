"""curvefp_quantize of fp32 rows whose workgroups take several rounds: both sides of the counts (4096 and 16384
rounds of 512 chunks) where the number of workgroups changes, a last one that is not full, a row stride.  Codes and
scales equal to those of the same rows quantized a few at a time, which are one round each."""

import pytest
import torch

from paper_2608_10010_amd import curvefp as cf
from tests.gpu_util import DEV, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["E4C3", "E5C2", "E3C3", "E4C3_r3/4"])
@pytest.mark.parametrize("rows,cols,pad", [(4096, 4096, 0), (4097, 4096, 0), (16384, 4096, 0), (16385, 4096, 8),
                                           (10001, 4128, 0), (20001, 4128, 0)])
def test_rounds(fmt, rows, cols, pad):
    say(f"[quantize rounds] {fmt} {rows} x {cols} + {pad}")
    g = torch.Generator(device=DEV).manual_seed(rows)
    x = torch.randn(rows, cols + pad, device=DEV, generator=g)[:, :cols]
    x *= torch.exp2(torch.randint(-20, 20, (rows, 1), device=DEV, generator=g).float())
    x[rows - 1, cols - 1] = float("nan")
    c, s = cf.curvefp_quantize(x, fmt)
    for r in range(0, rows, 1000):
        c2, s2 = cf.curvefp_quantize(x[r:r + 1000], fmt)
        assert torch.equal(c[r:r + 1000], c2) and torch.equal(s[r:r + 1000], s2), f"rows from {r}"
    assert int(s[rows - 1, -1]) == -128

"""Quantize-transpose tiles of 64 and 128 columns: column counts at the edges of both widths, one and several
tiles of 128 rows, both sides of the count of tiles (768 of 64 columns) from which bf16 sources take the form that
quantizes eight values at a time, a row stride, scales formed in the tile (G = 32) and given to it, blocks near the ends of
fp32's range and non-finite blocks; codes and scales equal to those of the transposed source quantized along
its rows."""

import pytest
import torch

from paper_2608_10010_amd import curvefp as cf
from tests.gpu_util import DEV, FMTS, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols,G", [(128, 8, 32), (128, 56, 32), (256, 64, 64), (128, 72, 32), (384, 120, 128),
                                         (128, 128, 32), (256, 136, 32), (256, 264, 64),
                                         (12288, 512, 32), (12288, 520, 32), (8192, 776, 64), (98432, 56, 32),
                                         (7168, 896, 32), (7168, 888, 64)])
def test_columns(fmt, dtype, rows, cols, G):
    say(f"[transpose tiles] {fmt} {dtype} {rows} x {cols} G={G}")
    g = torch.Generator(device=DEV).manual_seed(rows + cols)
    x = torch.randn(rows, cols + 8, device=DEV, generator=g)
    x *= torch.exp2(torch.randint(-20, 20, (rows, 1), device=DEV, generator=g).float())
    x[:, 0] *= 2.0 ** -110
    x[:32, 1] = 0
    x[5, cols // 2] = float("nan")
    x[rows - 1, cols - 1] = float("inf")
    x = x.to(dtype)[:, :cols]
    c, s = cf.curvefp_quantize(x, fmt, block_axis=0, block=G)
    c2, s2 = cf.curvefp_quantize(x.t().contiguous(), fmt, block=G)
    torch.cuda.synchronize()
    assert bool((s == s2).all()), f"{int((s != s2).sum())} scales differ"
    assert bool((c.reshape(-1) == c2.reshape(-1)).all()), f"{int((c.reshape(-1) != c2.reshape(-1)).sum())} bytes differ"

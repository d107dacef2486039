"""GPU parity of curvefp_quantize_compact's register kernel at its edges: both sides of each row length
rule (1024, 4096, 8192, 12288, 16384), rows that end inside a workgroup, blocks of the whole row, rows of zeros and
rows with nonfinite blocks."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_10010_amd import curvefp as cf
from paper_2608_10010_amd import workloads as W
from tests.gpu_util import FMTS, layout_codes, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,cols,G,S", [(5, 1024, 32, 4), (3, 1056, 32, 5), (7, 4096, 64, 5), (2, 4128, 32, 4),
                                           (3, 8192, 512, 5), (2, 8224, 32, 7), (2, 16384, 128, 5),
                                           (2, 16416, 32, 4), (6, 512, 512, 2), (1, 32, 32, 8),
                                           (3, 8448, 256, 5), (3, 15872, 512, 5), (2, 5120, 256, 3), (5, 768, 256, 4),
                                           (2, 12288, 256, 5), (2, 12320, 32, 4)])
def test_rows(dtype, rows, cols, G, S):
    rng = np.random.default_rng(rows * cols + G)
    x = (rng.standard_normal((rows, cols)) * np.exp2(rng.uniform(-20, 4, (rows, cols // 32)).repeat(32, 1)))
    x = x.astype(np.float32)
    x[rows - 1] = 0.0
    x[0, :G] = 0.0
    if rows > 2:
        x[1, cols - 1] = np.nan
    if dtype == "bf16":
        x = W.bf16_round(x)
    fmt = FMTS[(rows + cols // 32) % len(FMTS)]
    say(f"[compact rows] {rows}x{cols} G={G} S={S} {fmt} {dtype}")
    codes, ref, offs = cf.curvefp_quantize_compact(to_dev(x, dtype), fmt, G, S)
    torch.cuda.synchronize()
    oc, oref, od = oracle.quantize_compact(x, oracle.get_format(fmt), G, S)
    assert np.array_equal(ref.cpu().numpy(), oref)
    assert np.array_equal(offs.cpu().numpy(), oracle.pack_offsets(od, S))
    exp = layout_codes(oc, fmt)
    assert np.array_equal(codes.cpu().numpy().reshape(exp.shape), exp)

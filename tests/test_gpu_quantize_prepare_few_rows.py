"""curvefp_quantize_prepare on few rows: rows of 129 to 512 chunks of 8 take a workgroup each while both
operands together hold at most 4 tiles of 256 rows, and a wave each above that.  Both sides of that line and
of the row lengths, ragged rows and row counts: codes, scales, prepared bytes and reconstruction identical to
the three separate calls', and the codes, scales and reconstruction to the oracle's."""

import numpy as np
import pytest
import torch

from paper_2608_10010_amd import curvefp as cf
from tests.gpu_util import DEV, say, to_dev
from tests.test_gpu_quantize_prepare import fused_vs_separate, oracle_check, same_bytes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["E4C3", "E3C3"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,k", [(1, 1056), (3, 1024), (33, 4096), (257, 2080), (1024, 1056), (1025, 1056),
                                    (5, 4128)])
def test_few_rows(fmt, dtype, rows, k):
    rng = np.random.default_rng(rows + k)
    x = (rng.standard_normal((rows, k)) * np.exp2(rng.integers(-12, 12, (rows, 1)))).astype(np.float32)
    t = to_dev(x, dtype)
    codes, scales, _, d = fused_vs_separate(t, fmt, 32, "few rows")
    oracle_check(t.float().cpu().numpy(), fmt, 32, codes, scales, d, f"few rows {fmt} {rows} x {k}")


@pytest.mark.parametrize("ra,rb", [(256, 768), (257, 768), (1, 1)])
def test_pair_counts_both_operands(ra, rb):
    """A pair's rows are counted together; every output is the single calls', whichever kernel each takes."""
    say(f"[few rows] pair {ra} + {rb} rows")
    g = torch.Generator(device=DEV).manual_seed(ra)
    a, b = (torch.randn(r, 2048, device=DEV, generator=g).to(torch.bfloat16) for r in (ra, rb))
    pa, pb = cf.curvefp_quantize_prepare_pair(a, b, "E4C3", dequantize_a=True)
    sa = cf.curvefp_quantize_prepare(a, "E4C3", dequantize=True)
    sb = cf.curvefp_quantize_prepare(b, "E4C3")
    torch.cuda.synchronize()
    for got, want in ((pa, sa), (pb, sb)):
        for x, y in zip(got, want):
            if x is not None and y is not None:
                same_bytes(x, y, f"pair {ra} + {rb}")

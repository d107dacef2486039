"""GPU parity of curvefp_quantize_mse where its search can go wrong: candidates ruled out by the clipped
maximum alone, sums of zero (ties go to the first candidate), more winning blocks than a wave holds, a last
workgroup with a single block."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import FMTS, say
from tests.test_gpu_quantize_mse import run_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("G", [32, 64, 128])
def test_search(fmt, dtype, G):
    rng = np.random.default_rng(G + 10 * FMTS.index(fmt))
    x = rng.standard_normal((257, G)).astype(np.float32)      # one block per row: 256 and one more
    x[0::4, 0] = 8.0 * np.abs(x[0::4]).max(axis=1)             # a lone maximum: clipping it never pays
    x[1::4] = np.where(rng.random(x[1::4].shape) < 0.5, 0.97, 0.51) * 2.0   # clipping often pays
    f = oracle.get_format(fmt)
    c, s = oracle.quantize(x[2::4], f, G)
    x[2::4] = oracle.dequantize(c, s, f, G)                   # exactly representable: every sum at a_c is zero
    say(f"[quantize_mse] search fmt={fmt} dtype={dtype} G={G}")
    run_and_compare(x, fmt, dtype, 1, 8, f"search {fmt} {dtype} G={G}", block=G)
    run_and_compare(np.ascontiguousarray(x.T), fmt, dtype, 0, 8, f"search {fmt} {dtype} G={G} axis0", block=G)

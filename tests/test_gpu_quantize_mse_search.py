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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("G,candidates", [(32, 1), (32, 2), (64, 4), (96, 8)])
def test_candidates_above_and_ties(dtype, G, candidates):
    """Radix 2^(3/4): scales three apart share their levels.  Blocks of values near the levels of a scale whose top
    lies just under the block's maximum: the scale below ceil-absmax and the second above it reconstruct alike, and the
    one below, earlier in the order, wins; with one candidate the one above does.  Beside them blocks whose best scale is
    ceil-absmax or the first above it, and blocks at the ends of the scale range."""
    rng = np.random.default_rng(G + candidates)
    n = rng.integers(-31, 63, (771, G))
    n[:, 0] = 63
    x = np.exp2(3.0 * n / 32) * (1 + rng.uniform(-2.0 ** -8, 2.0 ** -8, n.shape))
    x[:, 0] = np.exp2(3.0 * 63 / 32) * (1 + 2.0 ** -7)
    x *= np.where(rng.random(n.shape) < 0.5, -1.0, 1.0)
    x[1::4] *= 2.0 ** -0.25                                   # off that scale's levels
    x[2::4, 0] *= 1.0 - 2.0 ** -5                             # the maximum under the top: ceil-absmax itself
    x[3::4, G // 2:] *= 2.0 ** -6                             # small values below the lower scales' range
    x *= np.exp2(rng.integers(-3, 4, (771, 1)))
    x[768] *= 2.0 ** -132                                     # subnormal maxima, and a maximum near fp32's
    x[769] *= 2.0 ** -125
    x[770] *= 2.0 ** 112
    say(f"[quantize_mse] above and ties dtype={dtype} G={G} candidates={candidates}")
    run_and_compare(x.astype(np.float32), "E4C3_r3/4", dtype, 1, candidates, f"ties {dtype} G={G}", block=G)

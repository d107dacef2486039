"""GPU parity of curvefp_quantize_tensorwise with more source units than the maximum pass has threads, the
maximum (or a NaN) in the last element, and the code buffer's first words, which carry the workgroups' maxima
between the passes, overwritten with codes."""

import numpy as np
import pytest

from tests.test_gpu_tensorwise import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,axis,shape", [("f32", 1, (4100, 2080)), ("bf16", 1, (4100, 2080)),
                                              ("bf16", 0, (2080, 4104)), ("f32", 0, (1056, 1001)),
                                              ("bf16", 1, (1, 32)), ("f32", 0, (32, 1))])
@pytest.mark.parametrize("last", [37.0, float("nan")])
def test_last_element(dtype, axis, shape, last):
    rng = np.random.default_rng(shape[0])
    x = np.clip(rng.standard_normal(shape), -4, 4).astype(np.float32)
    x[-1, -1] = last
    check(x, "E4C3" if axis else "E3C3", dtype, axis, f"last={last}")

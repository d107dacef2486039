"""GPU parity of curvefp_quantize_tensorwise with more source units than the maximum pass has threads, the
maximum (or a NaN) in the last element, and the code buffer's first words, which carry the workgroups' maxima
between the passes, overwritten with codes."""

import numpy as np
import pytest
import torch

from paper_2608_10010_amd import curvefp as cf
from tests.gpu_util import DEV, FMTS, say
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


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("dtype,rows,cols,axis", [(torch.float32, 8200, 4128, 1), (torch.bfloat16, 16400, 4128, 1),
                                                  (torch.bfloat16, 16416, 4128, 0), (torch.float32, 8224, 4100, 0)])
def test_streamed(fmt, dtype, rows, cols, axis):
    """More than 128 MiB, which both passes stream: codes equal to those of a few rows (columns) at a time, each with
    the tensor's largest value beside them, which are small tensors."""
    say(f"[tensorwise] streamed {fmt} {dtype} {rows} x {cols} axis={axis}")
    g = torch.Generator(device=DEV).manual_seed(rows)
    x = torch.randn(rows, cols, device=DEV, generator=g).clamp_(-4, 4).to(dtype)
    x[rows - 1, cols - 1] = 37.0
    assert x.numel() * x.element_size() > 128 << 20
    q, s = cf.curvefp_quantize_tensorwise(x, fmt, block_axis=axis)
    outer = rows if axis == 1 else cols
    for r in (0, 2048, outer - 300):
        part = x[r:r + 300] if axis == 1 else x[:, r:r + 300]
        extra = torch.zeros(*((1, cols) if axis == 1 else (rows, 4)), device=DEV, dtype=dtype)
        extra[0, 0] = 37.0
        q2, s2 = cf.curvefp_quantize_tensorwise(torch.cat((part, extra), dim=1 - axis).contiguous(), fmt, block_axis=axis)
        assert torch.equal(q[r:r + 300], q2[:300]), f"codes from {r}"
        assert torch.equal(s[r:r + 300], s2[:300])
    assert int(s.min()) == int(s.max())

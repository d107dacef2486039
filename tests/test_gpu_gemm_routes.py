"""Products of two formats, and outputs whose rows lie far apart, on each of the kernels that a product can take: the
small one (waves share K), 128 x 128 tiles with K in two halves, 256 x 256 tiles with K whole and in two halves.
`route` tells from what a call leaves in its workspace which one ran, so that a shape that a changed rule sends
elsewhere fails here."""

import numpy as np
import pytest
import torch

from paper_2608_10010_amd import curvefp as cf
from tests.gpu_util import DEV, FMTS, check_gemm, say, to_dev
from tests.test_gpu_gemm import oracle_gemm
from tests.test_gpu_gemm_mixed import gpu_operand, operand_source, oracle_mixed

pytestmark = pytest.mark.gpu


def route(M, N, K):
    """The kernel of an M x N x K product: "small" uses no workspace, 256 x 256 tiles with K in halves fill the slots
    at its end, 128 x 128 tiles with K in halves only the planes at its start; "whole": planes, and no slots."""
    a, b = (torch.ones(r, K, device=DEV) for r in (M, N))
    ws = torch.full((cf.curvefp_gemm_workspace_bytes(M, N, K),), 0xA5, dtype=torch.uint8, device=DEV)
    cf.curvefp_gemm_ws(*cf.curvefp_quantize(a, "E4C3"), *cf.curvefp_quantize(b, "E4C3"), M, N, K, "E4C3", workspace=ws)
    torch.cuda.synchronize()
    if bool((ws[:4096] == 0xA5).all()):
        return "small"
    tiles = -(-M // 256) * -(-N // 256)
    if tiles >= 256 or K < 512:
        return "whole"
    return "128 halves" if bool((ws[-4096:] == 0xA5).all()) else "256 halves"


def sample(rng, n, count):
    return np.unique(np.r_[0, n - 1, rng.integers(0, n, count)])


def two_formats(fa, fb, ta, tb, M, N, K):
    """gemm_mixed against the oracle on sampled rows and columns, and against the prepared operands bit for bit."""
    rng = np.random.default_rng(M + 31 * FMTS.index(fa) + 7 * FMTS.index(fb) + 2 * ta + tb)
    A = operand_source(rng, M, K, ta)
    B = operand_source(rng, N, K, tb, spread=3.0)
    qa, qb = gpu_operand(A, fa, "f32", 1), gpu_operand(B, fb, "f32", 1)
    C = cf.curvefp_gemm_mixed(*qa, fa, ta, *qb, fb, tb, M, N, K)
    pa, pb = cf.curvefp_prepare(*qa, M, K, fa, trans=ta), cf.curvefp_prepare(*qb, N, K, fb, trans=tb)
    Cp = cf.curvefp_gemm_prepared(pa, fa, pb, fb, M, N, K)
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int32), Cp.view(torch.int32)), "prepared operands differ"
    rows, cols = sample(rng, M, 12), sample(rng, N, 12)
    V, tol = oracle_mixed(A, fa, 1, ta, B, fb, 1, tb, rows, cols)
    return check_gemm(C.cpu().numpy()[np.ix_(rows, cols)], V, tol, f"{fa}x{fb} trans={ta}{tb} {M}x{N}x{K}")


LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]
LARGE = {(1056, 1056, 544): "128 halves", (2080, 4128, 96): "whole", (2080, 3104, 544): "256 halves"}


@pytest.mark.parametrize("shape", list(LARGE), ids=lambda s: "x".join(map(str, s)))
def test_pairs_on_large_tiles(shape):
    """Every pair of formats (the 256 x 256 kernel is compiled for each sum of their exponent offsets), the layouts in
    turn; each pair of two formats also with both operands along K."""
    say(f"[gemm routes] {shape}: {route(*shape)}")
    assert route(*shape) == LARGE[shape]
    worst = 0.0
    for i, (fa, fb) in enumerate((fa, fb) for fa in FMTS for fb in FMTS):
        for ta, tb in {(0, 0), LAYOUTS[i % 4]}:
            worst = max(worst, two_formats(fa, fb, ta, tb, *shape))
        say(f"[gemm routes] {shape} {fa} x {fb}")
    say(f"[gemm routes] {shape} worst rel_frob={worst:.2e}")


@pytest.mark.parametrize("fa,fb", [("E4C3", "E5C2"), ("E3C3", "E4C3"), ("E5C2", "E3C3"), ("E3C3", "E3C3")])
@pytest.mark.parametrize("shape", [(7, 6161, 1184), (33, 4097, 1056), (31, 12301, 2080), (500, 2000, 2080)],
                         ids=lambda s: "x".join(map(str, s)))
def test_two_formats_on_small_tiles(shape, fa, fb):
    """16 x 32, 32 x 32, 32 x 64 and 64 x 32 outputs per workgroup with a table for each operand."""
    say(f"[gemm routes] small {shape} {fa} x {fb}")
    assert route(*shape) == "small"
    two_formats(fa, fb, 0, 0, *shape)


WIDE = {(8, 40, 64): "small", (1100, 1000, 544): "128 halves", (2049, 3100, 544): "256 halves", (2049, 4100, 96): "whole"}


@pytest.mark.parametrize("shape", list(WIDE), ids=lambda s: "x".join(map(str, s)))
def test_very_wide_row_stride(shape):
    """Rows of C 4 MB apart (64-bit addresses), from the workspace and, where K is split there, with the halves added
    by atomics into a cleared C (curvefp_gemm); the gaps stay as they were."""
    M, N, K = shape
    ldc = (1 << 20) + 64
    need = M * ldc * 4
    free, _ = torch.cuda.mem_get_info()
    if free < need * 1.5:
        pytest.skip(f"needs {need / 2**30:.0f} GiB of free device memory, {free / 2**30:.0f} GiB free")
    assert route(*shape) == WIDE[shape]
    rng = np.random.default_rng(M)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((N, K)).astype(np.float32)
    say(f"[gemm routes] {shape} ldc={ldc}")
    qa, qb = cf.curvefp_quantize(to_dev(A, "f32"), "E4C3"), cf.curvefp_quantize(to_dev(B, "f32"), "E4C3")
    rows, cols = sample(rng, M, 12), sample(rng, N, 12)
    V, tol = oracle_gemm(A, B, "E4C3", rows=rows, cols=cols)
    dense = cf.curvefp_gemm_ws(*qa, *qb, M, N, K, "E4C3")
    check_gemm(dense.cpu().numpy()[np.ix_(rows, cols)], V, tol, f"{shape}")
    out = torch.empty((M, ldc), device=DEV)
    for call in (cf.curvefp_gemm_ws, cf.curvefp_gemm):
        out.fill_(3.0)
        call(*qa, *qb, M, N, K, "E4C3", c=out[:, :N])
        torch.cuda.synchronize()
        assert torch.equal(out[:, :N].contiguous().view(torch.int32), dense.view(torch.int32)), call.__name__
        assert float(out[:, N:].max()) == 3.0 and float(out[:, N:].min()) == 3.0, f"{call.__name__}: gaps written"

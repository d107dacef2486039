"""GPU parity of the three tile sizes a product can be computed with (16 TM x 16 TN with the waves
sharing K, 128 x 128, 256 x 256) at the sizes where they can go wrong: one element, edges of tiles and
fragments, remainders of the four-block groups and of the K halves, both sides of each size rule.

Sampled rows against the float64 product of the oracle's reconstructed values within the GEMM bound of
tests/gpu_util.gemm_tolerance, and every entry point against curvefp_gemm_ws bit for bit."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_10010_amd import curvefp as cf
from tests.gpu_util import FMTS, check_gemm, exact_values, gemm_tolerance, say, to_dev
from tests.test_gpu_gemm_mixed import oracle_mixed

pytestmark = pytest.mark.gpu

SHAPES = [
    # up to 2^20 outputs: waves share K
    (1, 1, 32), (16, 16, 128), (17, 15, 160), (33, 47, 288), (65, 129, 1056), (16, 4000, 96), (33, 4097, 96),
    (5000, 1, 32), (4097, 17, 160), (9, 40, 9248), (1024, 1024, 512),
    # the same, tiles of 16 x 32, 32 x 64 and 64 x 32 outputs, several groups of K blocks for each wave
    (7, 6161, 1184), (16, 11009, 1056), (31, 12301, 2080), (500, 2000, 2080),
    # no room for C in the workspace, and past the limit: 128 x 128 tiles, K whole
    (130, 2050, 64), (1024, 1024, 64), (1025, 1024, 96), (300, 4000, 480),
    # 128 x 128 tiles, K in two halves (of 8 and 8, 9 and 8, 17 and 16 blocks)
    (1025, 1024, 512), (300, 4000, 544), (1100, 1000, 1056),
    # 256 x 256 tiles, K whole and split
    (2049, 4100, 96), (2049, 3100, 544),
]


def sources(M, N, K, seed, poison):
    rng = np.random.default_rng(seed)
    A = (rng.standard_normal((M, K)) * np.exp2(rng.uniform(-6, 6, (M, 1)))).astype(np.float32)
    B = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    if K > 32:
        A[M // 2, :32] *= np.float32(2.0 ** -30)     # a block far below its row's top
        B[N // 3, K - 32:] *= np.float32(2.0 ** -27)
        A[M - 1, 32:64] = 0.0                        # an all-zero block
    if poison:
        A[M // 3, K - 1] = np.nan
        B[N - 1, K // 2] = np.inf
    return A, B


def run_shape(M, N, K, fmt, block, poison, dtype="f32"):
    A, B = sources(M, N, K, M + 3 * N + K, poison)
    qa = cf.curvefp_quantize(to_dev(A, dtype), fmt, block=block)
    qb = cf.curvefp_quantize(to_dev(B, dtype), fmt, block=block)
    out = torch.full((M, N + 4), 7.0, device="cuda")                       # a wider C: ldc > N
    Cw = cf.curvefp_gemm_ws(*qa, *qb, M, N, K, fmt, block=block)
    Cf = cf.curvefp_gemm(*qa, *qb, M, N, K, fmt, block=block, c=out)[:, :N].contiguous()
    Cm = cf.curvefp_gemm_mixed(qa[0], qa[1], fmt, 0, qb[0], qb[1], fmt, 0, M, N, K, block=block)
    pa, pb = cf.curvefp_prepare(*qa, M, K, fmt, block=block), cf.curvefp_prepare(*qb, N, K, fmt, block=block)
    Cp = cf.curvefp_gemm_prepared(pa, fmt, pb, fmt, M, N, K)
    torch.cuda.synchronize()
    assert bool((out[:, N:] == 7.0).all()), "columns past N written"
    for name, C in (("fused", Cf), ("mixed", Cm), ("prepared", Cp)):
        assert torch.equal(C.view(torch.int32), Cw.view(torch.int32)), f"{name} differs from ws"
    if N % 64 == 0:
        rq = cf.curvefp_gemm_requant(*qa, *qb, M, N, K, fmt, "E3C3", block=block, out_block=64)
        ref = cf.curvefp_quantize(Cw, "E3C3", block=64)
        assert torch.equal(rq[0], ref[0]) and torch.equal(rq[1], ref[1]), "requantized output"
    f = oracle.get_format(fmt)
    rows = np.unique(np.r_[0, M // 3, M // 2, M - 1, np.arange(0, M, max(1, M // 5))])
    ca, sa = oracle.quantize(A[rows], f, block)
    cb, sb = oracle.quantize(B, f, block)
    V = exact_values(ca, sa, fmt, block) @ exact_values(cb, sb, fmt, block).T
    V[(sa == oracle.POISON_SCALE).any(axis=1)] = np.nan
    V[:, (sb == oracle.POISON_SCALE).any(axis=1)] = np.nan
    return check_gemm(Cw.cpu().numpy()[rows], V, gemm_tolerance(ca, sa, cb, sb, fmt, block), f"{fmt} {M}x{N}x{K}")


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_shapes(shape):
    M, N, K = shape
    fmt = FMTS[(M + N) % len(FMTS)]
    block = 64 if K % 64 == 0 and M % 2 else 32
    say(f"[tiles] {M}x{N}x{K} {fmt} G={block}")
    say(f"[tiles] rel_frob={run_shape(M, N, K, fmt, block, False):.2e}")


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("shape", [(40, 72, 416), (1030, 1100, 544), (2049, 3100, 544)],
                         ids=lambda s: "x".join(map(str, s)))
def test_formats_with_nonfinite_blocks(shape, fmt):
    """Every format on every tile size, one row and one column poisoned."""
    say(f"[tiles] poisoned {shape} {fmt}")
    run_shape(*shape, fmt, 32, True)


@pytest.mark.parametrize("shape", [(96, 160, 352), (1056, 1024, 544)], ids=lambda s: "x".join(map(str, s)))
def test_two_formats_and_reused_operand(shape):
    """E5C2 along K times reused E4C3 codes ([K][N], blocks along N): the mixed call and prepared operands
    agree bit for bit, sampled rows with the oracle."""
    M, N, K = shape
    rng = np.random.default_rng(M)
    A = rng.standard_normal((M, K)).astype(np.float32)
    X = (rng.standard_normal((K, N)) * 0.5).astype(np.float32)
    say(f"[tiles] mixed {shape}")
    qa, qx = cf.curvefp_quantize(to_dev(A, "f32"), "E5C2"), cf.curvefp_quantize(to_dev(X, "f32"), "E4C3")
    C = cf.curvefp_gemm_mixed(*qa, "E5C2", 0, *qx, "E4C3", 1, M, N, K)
    pa, px = cf.curvefp_prepare(*qa, M, K, "E5C2"), cf.curvefp_prepare(*qx, N, K, "E4C3", trans=1)
    Cp = cf.curvefp_gemm_prepared(pa, "E5C2", px, "E4C3", M, N, K)
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int32), Cp.view(torch.int32))
    rows = np.arange(0, M, max(1, M // 6))
    V, tol = oracle_mixed(A[rows], "E5C2", 1, 0, X, "E4C3", 1, 1)
    check_gemm(C.cpu().numpy()[rows], V, tol, f"mixed {shape}")

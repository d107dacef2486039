"""curvefp_gemm_requant where K is split in two: the 256 x 256 tiles' halves are added and quantized from their
slots by a kernel of its own, the 128 x 128 tiles' C is quantized from the workspace.  Rows that end inside a
wave's eight, columns that end inside a tile, every output format, output blocks of 32 to 256 and poisoned
rows and columns: codes and scales equal to curvefp_quantize of curvefp_gemm_ws's C, bit for bit."""

import numpy as np
import pytest
import torch

from paper_2608_10010_amd import curvefp as cf
from tests.gpu_util import DEV, FMTS, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ofmt", FMTS)
@pytest.mark.parametrize("M,N,K,G", [(1500, 4000, 640, 32), (1537, 3840, 512, 256), (1501, 3968, 544, 64),   # slots
                                     (520, 3840, 640, 32), (777, 2816, 544, 256)])             # 128 x 128 tiles
@pytest.mark.parametrize("poison", [False, True])
def test_split_requant(ofmt, M, N, K, G, poison):
    say(f"[requant slots] -> {ofmt} M={M} N={N} K={K} G={G} poison={poison}")
    rng = np.random.default_rng(M + G)
    A = (rng.standard_normal((M, K)) * np.exp2(rng.uniform(-4, 4, (M, 1)))).astype(np.float32)
    B = (rng.standard_normal((N, K)) * 0.05).astype(np.float32)
    if poison:
        A[M - 1, 3] = np.nan
        A[17, K - 1] = np.inf
        B[N - 1, 0] = np.nan
        A[40:48] = 0.0
    ca, sa = cf.curvefp_quantize(to_dev(A, "f32"), "E4C3")
    cb, sb = cf.curvefp_quantize(to_dev(B, "f32"), "E4C3")
    ws = cf.gemm_workspace(M, N, K, DEV)
    codes, scales = cf.curvefp_gemm_requant(ca, sa, cb, sb, M, N, K, "E4C3", ofmt, workspace=ws, out_block=G)
    C = cf.curvefp_gemm_ws(ca, sa, cb, sb, M, N, K, "E4C3", workspace=ws)
    c2, s2 = cf.curvefp_quantize(C, ofmt, block=G)
    torch.cuda.synchronize()
    assert bool((scales == s2).all()), f"{int((scales != s2).sum())} scales differ"
    a, b = codes.reshape(-1), c2.reshape(-1)
    assert a.numel() == b.numel() and bool((a == b).all()), f"{int((a != b).sum())} code bytes differ"
    if poison:
        assert bool((scales[M - 1] == -128).all()) and bool((scales[:, -1] == -128).all())


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("M,N,K,G", [(1500, 3840, 544, 64), (2049, 4128, 96, 32), (2049, 4224, 64, 128)])
def test_input_formats(fmt, M, N, K, G):
    """Every input format (the requantizing 256 x 256 kernel is compiled for each one's exponent offset), K in halves
    and whole, where the tile is quantized in the epilogue: every output format."""
    rng = np.random.default_rng(M + G)
    A = (rng.standard_normal((M, K)) * np.exp2(rng.uniform(-4, 4, (M, 1)))).astype(np.float32)
    B = (rng.standard_normal((N, K)) * 0.05).astype(np.float32)
    ca, sa = cf.curvefp_quantize(to_dev(A, "f32"), fmt)
    cb, sb = cf.curvefp_quantize(to_dev(B, "f32"), fmt)
    ws = cf.gemm_workspace(M, N, K, DEV)
    C = cf.curvefp_gemm_ws(ca, sa, cb, sb, M, N, K, fmt)
    for ofmt in FMTS:
        say(f"[requant slots] {fmt} -> {ofmt} M={M} N={N} K={K} G={G}")
        codes, scales = cf.curvefp_gemm_requant(ca, sa, cb, sb, M, N, K, fmt, ofmt, workspace=ws, out_block=G)
        c2, s2 = cf.curvefp_quantize(C, ofmt, block=G)
        torch.cuda.synchronize()
        assert torch.equal(scales, s2) and torch.equal(codes.reshape(-1), c2.reshape(-1)), f"{fmt} -> {ofmt}"

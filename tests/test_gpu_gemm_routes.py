"""Every kernel that a product can take (the small one, whose waves share K; 128 x 128 tiles with K in two halves; 256 x
256 tiles with K whole and in two halves) on what the other files test at sizes that one of them takes: pairs of
formats, rows of C far apart, edge operands, the accuracy contract, block sizes, a workspace's contents, capture, long K.
`route` tells from what a call leaves in its workspace which one ran, so that a shape that a changed rule sends
elsewhere fails here."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_10010_amd import curvefp as cf
from paper_2608_10010_amd import workloads as W
from tests import test_gpu_accuracy_contract as contract
from tests.gpu_util import DEV, FMTS, check_gemm, gemm_tolerance, say, to_dev
from tests.test_gpu_gemm import EDGE_PAIRS, oracle_gemm
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


# ---------------------------------------------------------------- the large tiles' own edges

# K = 512 and more: in two halves on 128 x 128 and on 256 x 256 tiles (rows and columns that end inside tiles)
SPLIT = {"128 halves": (1100, 1030), "256 halves": (2049, 3100)}


def every_call(qa, qb, M, N, K, fmt, G=32):
    """C of curvefp_gemm_ws, after the other entry points gave the same bits."""
    C = cf.curvefp_gemm_ws(*qa, *qb, M, N, K, fmt, block=G)
    pa, pb = cf.curvefp_prepare(*qa, M, K, fmt, block=G), cf.curvefp_prepare(*qb, N, K, fmt, block=G)
    others = {"fused": cf.curvefp_gemm(*qa, *qb, M, N, K, fmt, block=G),
              "prepared": cf.curvefp_gemm_prepared(pa, fmt, pb, fmt, M, N, K),
              "mixed": cf.curvefp_gemm_mixed(*qa, fmt, 0, *qb, fmt, 0, M, N, K, block=G)}
    torch.cuda.synchronize()
    for name, X in others.items():
        assert torch.equal(X.view(torch.int32), C.view(torch.int32)), f"{name} differs from ws"
    return C.cpu().numpy()


def repeat_to(x, rows):
    return np.ascontiguousarray(np.tile(x, (-(-rows // x.shape[0]), 1))[:rows])


@pytest.mark.parametrize("kind", list(EDGE_PAIRS))
@pytest.mark.parametrize("tiles", list(SPLIT))
def test_edges_on_large_tiles(kind, tiles):
    """The edge operands of test_gpu_gemm, their 96 and 80 rows repeated over the large tiles, one format each."""
    (M, N), K = SPLIT[tiles], 544
    fmt = FMTS[list(EDGE_PAIRS).index(kind) % len(FMTS)]
    ka, kb = EDGE_PAIRS[kind]
    A, B = W.edge_tensor(ka, (96, K), seed=21), W.edge_tensor(kb, (80, K), seed=22)
    if kind == "wide_range":
        A = (A * np.float32(2.0 ** -4)).astype(np.float32)
    say(f"[gemm routes] edges {kind} {fmt} {tiles}")
    assert route(M, N, K) == tiles
    q = [cf.curvefp_quantize(to_dev(repeat_to(X, R), "f32"), fmt) for X, R in ((A, M), (B, N))]
    C = every_call(*q, M, N, K, fmt)
    V, tol = oracle_gemm(A, B, fmt)
    i, j = np.arange(M) % 96, np.arange(N) % 80
    check_gemm(C, V[np.ix_(i, j)], tol[np.ix_(i, j)], f"{fmt} {kind} {tiles}")


@pytest.mark.parametrize("fmt", ["E4C3", "E5C2", "E3C3"])
@pytest.mark.parametrize("tiles", list(SPLIT))
def test_accuracy_contract_on_large_tiles(fmt, tiles):
    """The clauses of test_gpu_accuracy_contract: rows of narrow scales without any loss, blocks 60 binades below their
    row's top flushed, blocks 20 to 36 below within the bound of what they may lose."""
    (M, N), K = SPLIT[tiles], contract.K
    f = oracle.get_format(fmt)
    rng = np.random.default_rng(75)
    m, n, nb = 48, 40, K // 32
    i, j = np.arange(M) % m, np.arange(N) % n
    assert route(M, N, K) == tiles
    for clause in ("narrow", "flush", "band"):
        say(f"[gemm routes] contract {clause} {fmt} {tiles}")
        ca, cb = contract.random_codes(rng, f, (m, K)), contract.random_codes(rng, f, (n, K))
        sb = rng.integers(-4, 4, (n, nb)).astype(np.int8)
        if clause == "narrow":
            sa = (rng.integers(-30, 30, (m, 1)) - rng.integers(0, 13, (m, nb))).astype(np.int8)
        else:
            sa = (10 - (rng.integers(20, 37, (m, nb)) if clause == "band" else np.full((m, nb), 60))).astype(np.int8)
            sa[:, 0] = 10
        if clause == "flush":
            cb[: n // 2, :32] = 0
        C = contract.gpu_gemms(repeat_to(ca, M), repeat_to(sa, M), repeat_to(cb, N), repeat_to(sb, N), fmt)
        for r in (slice(0, m), slice(M - m, M)):              # the first and the last rows and columns whole
            for c in (slice(0, n), slice(N - n, N)):
                ii, jj = i[r], j[c]
                V = oracle.gemm_exact(ca[ii], sa[ii], cb[jj], sb[jj], f)
                args = (ca[ii], sa[ii], cb[jj], sb[jj], fmt)
                if clause == "narrow":
                    contract.strict(C[r, c], V, *args, f"narrow {fmt} {tiles}")
                check_gemm(C[r, c], V, gemm_tolerance(*args), f"{clause} {fmt} {tiles}", frobenius=clause == "narrow")
                if clause == "flush":
                    assert np.all(C[r, c][:, jj < n // 2] == 0) and np.all(np.abs(V[:, jj < n // 2]) > 0)
        # every repetition of a row and column is the same product
        first = C[:m, :n]
        assert np.array_equal(C, first[np.ix_(i, j)]), f"{clause} {fmt} {tiles}: repetitions differ"


@pytest.mark.parametrize("fmt", ["E4C3", "E3C3", "E4C3_r3/4"])
@pytest.mark.parametrize("K,G", [(576, 64), (576, 96), (1024, 512), (544, 544), (96, 96)])
@pytest.mark.parametrize("tiles", list(SPLIT))
def test_block_sizes_on_large_tiles(fmt, K, G, tiles):
    """Blocks of G (K = 96: K whole): every entry point agrees, and with the same codes at scales repeated per 32."""
    M, N = SPLIT[tiles] if K >= 512 else (1100, 1030) if tiles == "128 halves" else (2049, 4100)
    rng = np.random.default_rng(K + G)
    A = (rng.standard_normal((M, K)) * np.exp2(rng.uniform(-8, 8, (M, 1)))).astype(np.float32)
    A[:, :32] *= np.float32(2.0 ** -9)
    B = rng.standard_normal((N, K)).astype(np.float32)
    say(f"[gemm routes] G={G} K={K} {fmt} {tiles}")
    assert route(M, N, K) == (tiles if K >= 512 else "whole")
    qa, qb = (cf.curvefp_quantize(to_dev(X, "f32"), fmt, block=G) for X in (A, B))
    C = every_call(qa, qb, M, N, K, fmt, G)
    ra, rb = ((q[0], torch.repeat_interleave(q[1], G // 32, dim=1).contiguous()) for q in (qa, qb))
    assert np.array_equal(C.view(np.uint32), every_call(ra, rb, M, N, K, fmt).view(np.uint32))


@pytest.mark.parametrize("tiles", list(SPLIT) + ["whole"])
def test_workspace_contents_do_not_matter(tiles):
    """Every call that takes a workspace gives the same bits three times over: on a workspace of one bits (counters,
    NaN sums), on what a larger product of other operands left there, and on its own leavings."""
    M, N, K = (*SPLIT[tiles], 544) if tiles in SPLIT else (2049, 4100, 96)
    fmt = "E4C3"
    g = torch.Generator(device=DEV).manual_seed(M)
    mk = lambda r: cf.curvefp_quantize(torch.randn(r, K, device=DEV, generator=g), fmt)
    qa, qb, la, lb = mk(M), mk(N), mk(M + 256), mk(N + 256)
    bt = cf.curvefp_quantize(torch.randn(K, N // 32 * 32, device=DEV, generator=g), fmt)
    pa, pb = cf.curvefp_prepare(*qa, M, K, fmt), cf.curvefp_prepare(*qb, N, K, fmt)
    ws = torch.empty(cf.curvefp_gemm_mixed_workspace_bytes(M + 256, N + 256, K), dtype=torch.uint8, device=DEV)
    Nt, Nq = N // 32 * 32, N // 64 * 64
    calls = {
        "ws": lambda: [cf.curvefp_gemm_ws(*qa, *qb, M, N, K, fmt, workspace=ws)],
        "prepared": lambda: [cf.curvefp_gemm_prepared(pa, fmt, pb, fmt, M, N, K, workspace=ws)],
        "mixed": lambda: [cf.curvefp_gemm_mixed(*qa, fmt, 0, *bt, fmt, 1, M, Nt, K, workspace=ws)],
        "requant": lambda: list(cf.curvefp_gemm_requant(*qa, qb[0][:Nq], qb[1][:Nq], M, Nq, K, fmt, "E5C2", workspace=ws,
                                                        out_block=64)),
    }
    say(f"[gemm routes] workspace contents {tiles}")
    assert route(M, N, K) == tiles
    for name, call in calls.items():
        got = []
        for left in ("one bits", "a larger product", "its own"):
            if left == "one bits":
                ws.fill_(0xFF)
            elif left == "a larger product":
                cf.curvefp_gemm_ws(*la, *lb, M + 256, N + 256, K, fmt, workspace=ws)
            got.append([t.clone() for t in call()])
        torch.cuda.synchronize()
        for other in got[1:]:
            assert all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(got[0], other)), name
        if name == "ws":
            ref = cf.curvefp_gemm(*qa, *qb, M, N, K, fmt)
            assert torch.equal(ref.view(torch.int32), got[0][0].view(torch.int32))
            if cf.curvefp_gemm_workspace_bytes(M, N, K) <= 128 << 20:
                st = cf.curvefp_gemm_ws_static(*qa, *qb, M, N, K, fmt)
                assert torch.equal(st.view(torch.int32), ref.view(torch.int32)), "static scratch"


@pytest.mark.parametrize("tiles", list(SPLIT))
def test_captured_calls_replay(tiles):
    """Products with K in halves and their requantized form in a captured graph, replayed on new operands with eager
    calls of the same kind in between: counters and slots are cleared or rewritten by each replay itself."""
    (M, N), K, fmt = SPLIT[tiles], 544, "E3C3"
    Nq = N // 64 * 64
    x, w = torch.empty(M, K, device=DEV, dtype=torch.bfloat16), torch.empty(N, K, device=DEV, dtype=torch.bfloat16)
    g = torch.Generator(device=DEV)

    def fill(seed):
        g.manual_seed(seed)
        x.copy_(torch.randn(M, K, device=DEV, generator=g))
        w.copy_(torch.randn(N, K, device=DEV, generator=g))

    def buffers():
        b = dict(qa=cf.curvefp_quantize(x, fmt), qb=cf.curvefp_quantize(w, fmt))
        b["pa"], b["pb"] = cf.curvefp_prepare(*b["qa"], M, K, fmt), cf.curvefp_prepare(*b["qb"], N, K, fmt)
        b["ws"] = cf.gemm_workspace(M, N, K, DEV)
        b["c"] = [torch.empty(M, N, device=DEV) for _ in range(2)]
        b["out"] = (torch.empty(M, Nq // 32, 28, dtype=torch.uint8, device=DEV),
                    torch.empty(M, Nq // 64, dtype=torch.int8, device=DEV))
        return b

    def step(b):
        cf.curvefp_quantize(x, fmt, codes=b["qa"][0], scales=b["qa"][1])
        cf.curvefp_quantize(w, fmt, codes=b["qb"][0], scales=b["qb"][1])
        cf.curvefp_gemm_ws(*b["qa"], *b["qb"], M, N, K, fmt, c=b["c"][0], workspace=b["ws"])
        cf.curvefp_prepare(*b["qa"], M, K, fmt, prepared=b["pa"])
        cf.curvefp_prepare(*b["qb"], N, K, fmt, prepared=b["pb"])
        cf.curvefp_gemm_prepared(b["pa"], fmt, b["pb"], fmt, M, N, K, c=b["c"][1], workspace=b["ws"])
        cf.curvefp_gemm_requant(*b["qa"], b["qb"][0][:Nq], b["qb"][1][:Nq], M, Nq, K, fmt, fmt, workspace=b["ws"],
                                out_block=64, out_codes=b["out"][0], out_scales=b["out"][1])

    fill(1)
    assert route(M, N, K) == tiles
    cap, eager = buffers(), buffers()
    step(cap)
    torch.cuda.synchronize()
    say(f"[gemm routes] capture {tiles}")
    graph, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=s):
        step(cap)
    for seed in (2, 3, 4):
        fill(seed)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        step(eager)
        torch.cuda.synchronize()
        for a, b in zip((*cap["qa"], *cap["c"], *cap["out"]), (*eager["qa"], *eager["c"], *eager["out"])):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), f"replay {seed}"
        assert torch.equal(cap["c"][0].view(torch.int32), cap["c"][1].view(torch.int32))


@pytest.mark.parametrize("tiles", list(SPLIT))
def test_long_k_on_large_tiles(tiles):
    """K = 2^18: planes of more than 2^31 bytes (256 x 256 tiles) under 64-bit block offsets."""
    (M, N), K, fmt = SPLIT[tiles], 1 << 18, "E5C2"
    need = 3 * (M + N + 512) * K * 4
    free, _ = torch.cuda.mem_get_info()
    if free < need * 1.2:
        pytest.skip(f"needs {need / 2**30:.0f} GiB of free device memory, {free / 2**30:.0f} GiB free")
    g = torch.Generator(device=DEV).manual_seed(M)
    x, w = (torch.randn(r, K, device=DEV, generator=g, dtype=torch.bfloat16) for r in (M, N))
    say(f"[gemm routes] K = 2^18 {tiles}")
    assert route(M, N, 544) == tiles                       # the rule beyond 512 does not depend on K
    qa, qb = cf.curvefp_quantize(x, fmt), cf.curvefp_quantize(w, fmt)
    Cw = cf.curvefp_gemm_ws(*qa, *qb, M, N, K, fmt)
    Cf = cf.curvefp_gemm(*qa, *qb, M, N, K, fmt)
    torch.cuda.synchronize()
    assert torch.equal(Cw.view(torch.int32), Cf.view(torch.int32))
    rows, cols = np.array([0, M // 2, M - 1]), np.array([0, 255, N - 1])
    A, B = (t[torch.from_numpy(i).to(DEV)].float().cpu().numpy() for t, i in ((x, rows), (w, cols)))
    V, tol = oracle_gemm(A, B, fmt)
    check_gemm(Cw.cpu().numpy()[np.ix_(rows, cols)], V, tol, f"K = 2^18 {tiles}", frobenius=False)

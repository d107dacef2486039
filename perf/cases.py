"""Performance cases of the CurveFP path: the calls a program makes, at the sizes it makes them.

Each case is a dict of plain values whose "kind" names a sequence of entry points of
``paper_2608_10010_amd.curvefp``; buffers, workspaces and weights that a program keeps from call
to call are made in ``prepare``, everything that depends on the pass's own tensors runs in
``run``.  The kinds:

linear      an activation quantized and multiplied by weight codes (the compact inference layer)
prepared    the same with the weight expanded once (static weights) and the activation quantized
            and expanded in one launch
requant     a linear layer whose output leaves as codes for the next one
step        both operands quantized and expanded in one launch, the activation reconstructed,
            then the product (weights that change from step to step)
forward     a training forward pass: activation along its rows, weight held K x N and quantized
            through the transpose, then the product
backward    a training backward pass: the output gradient quantized once, then both products with
            the codes kept from the forward pass
roundtrip   quantize and reconstruct (blocks along the rows)
mse         weights quantized offline with searched scales
compact     S-bit scale exponents: quantize, unpack the scales, reconstruct
tensorwise  one scale for the tensor
"""

import math

import torch

from paper_2608_10010_amd import curvefp as cf

# ---------------------------------------------------------------- formats (for `exact` and sizes)

# name: (C, n_max, p, q): levels 2^(p n / (q 2^C)), n in [-n_max, n_max]
_FMT = {
    "E4C3": (3, 63, 1, 1),
    "E5C2": (2, 63, 1, 1),
    "E3C3": (3, 31, 1, 1),
    "E4C3_r8/9": (3, 63, 8, 9),
    "E4C3_r3/4": (3, 63, 3, 4),
}


def _code_bytes(fmt, n):
    return n * 7 / 8 if fmt == "E3C3" else n


# ---------------------------------------------------------------- cases

def listed():
    return [
        # the smallest call: a 128-cube layer on fp32 tensors, where launches and host time count
        dict(name="tiny", kind="linear", fmt="E4C3", block=32, dtype="f32", M=128, N=128, K=128),
        # decode: one batch of 16 tokens through a 4096 x 4096 layer of CurveFP7 weight codes
        dict(name="decode", kind="linear", fmt="E3C3", block=32, dtype="bf16", M=16, N=4096, K=4096),
        # decode with the weights of a gate/up projection held expanded
        dict(name="decode_prepared", kind="prepared", fmt="E4C3", block=32, dtype="bf16", M=32, N=14336, K=4096),
        # a short ragged prompt through a QKV projection, blocks of 64
        dict(name="prompt_ragged", kind="linear", fmt="E4C3", block=64, dtype="bf16", M=333, N=6144, K=4096),
        # prefill of 2048 tokens, the compact inference layer, output handed on as codes
        dict(name="prefill_requant", kind="requant", fmt="E3C3", block=32, dtype="bf16", M=2048, N=4096, K=4096,
             out_fmt="E3C3", out_block=64),
        # a 7B up-projection's training forward pass on 4096 tokens
        dict(name="forward", kind="forward", fmt="E4C3", block=32, dtype="bf16", M=4096, N=11008, K=4096),
        # its backward pass (dX and dW) from E5C2 gradients and the forward pass's E4C3 codes
        dict(name="backward", kind="backward", fmt="E5C2", fmt_b="E4C3", block=32, dtype="bf16", M=4096, N=11008,
             K=4096),
        # the largest: the 8B gate/up projection on 8192 tokens, both operands new
        dict(name="step_gateup", kind="step", fmt="E4C3", block=32, dtype="bf16", M=8192, N=14336, K=4096),
        # fp32 gradients quantized and reconstructed, rows taken out of a wider buffer
        dict(name="roundtrip_f32", kind="roundtrip", fmt="E5C2", block=32, dtype="f32", M=4000, K=11008, pad=64),
        # offline weight quantization at the paper's post-training block of 64
        dict(name="weights_mse", kind="mse", fmt="E3C3", block=64, dtype="bf16", M=4096, K=4096, candidates=4),
        # cached activations with 5-bit scale exponents in blocks of 64
        dict(name="compact_acts", kind="compact", fmt="E3C3", block=64, dtype="bf16", M=2048, K=4096, bits=5),
        # one scale for a weight of odd width, the rational radix
        dict(name="tensorwise_odd", kind="tensorwise", fmt="E4C3_r3/4", block=32, dtype="bf16", M=1511, K=5152),
    ]


_MAX_FLOPS = 2.0 * 8192 * 14336 * 4096


def draw(rng):
    """One more case of the ranges above: kinds, formats, types, blocks and (log-uniform) sizes."""
    def size(lo, hi, step=1):
        v = math.exp(rng.uniform(math.log(lo), math.log(hi + step)))
        return int(min(hi, max(lo, int(v / step) * step)))

    kind = rng.choice(["linear", "linear", "prepared", "requant", "step", "forward", "backward", "roundtrip", "mse",
                       "compact", "tensorwise"])
    block = rng.choice([32, 32, 32, 64, 128])
    fmt = rng.choice(["E4C3", "E4C3", "E5C2", "E3C3", "E3C3", "E4C3_r8/9", "E4C3_r3/4"])
    c = dict(kind=kind, fmt=fmt, block=block, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))
    if kind in ("linear", "prepared"):
        c.update(M=size(1, 4096), N=size(64, 14336), K=size(128, 14336, block))
    elif kind == "requant":
        ob = rng.choice([32, 64, 128, 256])
        c.update(M=size(16, 4096), N=size(256, 14336, ob), K=size(256, 14336, block),
                 out_fmt=rng.choice(["E3C3", "E4C3"]), out_block=ob)
    elif kind == "step":
        c.update(M=size(256, 8192), N=size(512, 14336), K=size(512, 14336, block))
    elif kind == "forward":
        c.update(M=size(256, 8192), N=size(512, 14336), K=size(512, 8192, block))
    elif kind == "backward":
        c.update(fmt="E5C2", fmt_b=rng.choice(["E4C3", "E3C3"]), M=size(256, 4096, block), N=size(512, 11008, block),
                 K=size(512, 4096, block))
    elif kind == "mse":
        c.update(M=size(64, 8192), K=size(256, 8192, block), candidates=rng.choice([2, 4, 6]))
    elif kind == "compact":
        c.update(M=size(16, 8192), K=size(256, 14336, block), bits=rng.choice([4, 5]))
    else:
        c.update(M=size(1, 16384), K=size(128, 14336, block))
        if kind == "roundtrip":
            c["pad"] = rng.choice([0, 0, 64])
    # nothing costs more than the largest listed case: fewer rows where the product is larger
    if "N" in c:
        per_row = (2 if kind == "backward" else 1) * 2.0 * c["N"] * c["K"]
        step = block if kind == "backward" else 1
        c["M"] = max(step, min(c["M"], int(_MAX_FLOPS / per_row) // step * step))
    return c


# ---------------------------------------------------------------- inputs

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed, salt):
    g = torch.Generator(device=_device())
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _randn(shape, g):
    return torch.randn(shape, generator=g, device=_device(), dtype=torch.float32)


def _activation(rows, cols, seed, dtype):
    """0.5 t(4) with 0.1% of the channels 20 times larger (outlier channels)."""
    g = _gen(seed, 1)
    x = _randn((rows, cols), g)
    chi = torch.zeros_like(x)
    for _ in range(4):
        chi += _randn((rows, cols), g).square_()
    x.mul_(0.5).div_(chi.mul_(0.25).sqrt_())
    ch = torch.randperm(cols, generator=g, device=_device())[:max(1, round(0.001 * cols))]
    x[:, ch] *= 20.0
    return x.to(_DT[dtype])


def _normal(rows, cols, seed, dtype, std, salt=2):
    return _randn((rows, cols), _gen(seed, salt)).mul_(std).to(_DT[dtype])


def _gradient(rows, cols, seed, dtype):
    """N(0, 1) with a scale of its own, exp(N(0, 3)), for each row (token)."""
    g = _gen(seed, 3)
    return (_randn((rows, cols), g) * torch.exp(3.0 * _randn((rows, 1), g))).to(_DT[dtype])


def _sources(c, seed):
    """The pass's own tensors: x, and w where the weight belongs to the pass or is kept as codes."""
    kind, M, K, dt = c["kind"], c["M"], c["K"], c["dtype"]
    if kind in ("linear", "prepared", "requant"):
        return _activation(M, K, seed, dt), _normal(c["N"], K, seed, dt, 0.02)
    if kind == "step":
        return _normal(M, K, seed, dt, 1.0, 4), _normal(c["N"], K, seed, dt, 0.02)
    if kind == "forward":                      # weight held K x N
        n = -(-c["N"] // 8) * 8                # rows of whole 16-byte pieces
        return _normal(M, K, seed, dt, 1.0, 4), _normal(K, n, seed, dt, 0.02)[:, :c["N"]]
    if kind == "backward":                     # dY [M][N]; forward X [M][K], W [K][N]
        return _gradient(M, c["N"], seed, dt), (_normal(M, K, seed, dt, 1.0, 4), _normal(K, c["N"], seed, dt, 0.02))
    if kind == "roundtrip":
        return _gradient(M, K + c.get("pad", 0), seed, dt)[:, :K], None
    if kind == "compact":
        return _activation(M, K, seed, dt), None
    return _normal(M, K, seed, dt, 0.02), None  # mse, tensorwise: weights


# ---------------------------------------------------------------- prepare and run

def _codes(fmt, rows, k):
    shape = (rows, k // 32, 28) if fmt == "E3C3" else (rows, k)
    return torch.empty(shape, dtype=torch.uint8, device="cuda")


def _scales(rows, n):
    return torch.empty((rows, n), dtype=torch.int8, device="cuda")


def _f32(rows, cols):
    return torch.empty((rows, cols), dtype=torch.float32, device="cuda")


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n > 0 else None


def prepare(case, seed):
    c = dict(case)
    kind, fmt, G, M, K = c["kind"], c["fmt"], c["block"], c["M"], c["K"]
    x, w = _sources(c, seed)
    s = dict(c=c, x=x)
    if kind == "backward":
        N = c["N"]
        xf, wf = w
        s["x_codes"] = cf.curvefp_quantize(xf, c["fmt_b"], block=G)                  # [M][K] along K
        s["w_codes"] = cf.curvefp_quantize(wf, c["fmt_b"], block_axis=0, block=G)    # [N][K] along K
        s["codes"], s["scales"] = _codes(fmt, M, N), _scales(M, N // G)
        s["dx"], s["dw"] = _f32(M, K), _f32(N, K)
        s["ws"] = _bytes(max(cf.curvefp_gemm_mixed_workspace_bytes(M, K, N),
                             cf.curvefp_gemm_mixed_workspace_bytes(N, K, M)))
        return s
    s["codes"] = _codes(fmt, M, K)
    if kind == "tensorwise":
        s["scales"], s["ws"] = _scales(M, 1), torch.empty(1, dtype=torch.int32, device="cuda")
        return s
    if kind == "compact":
        s["ref"] = torch.empty(M, dtype=torch.int8, device="cuda")
        s["offsets"] = torch.empty((M, cf.curvefp_compact_offsets_bytes(1, K, G, c["bits"])), dtype=torch.uint8,
                                   device="cuda")
    s["scales"] = _scales(M, K // G)
    if kind in ("roundtrip", "compact"):
        s["dst"] = _f32(M, K)
    if kind in ("linear", "requant"):
        s["w_codes"] = cf.curvefp_quantize(w, fmt, block=G)
        s["ws"] = _bytes(cf.curvefp_gemm_workspace_bytes(M, c["N"], K))
    if kind == "requant":
        s["out"] = (_codes(c["out_fmt"], M, c["N"]), _scales(M, c["N"] // c["out_block"]))
    if kind in ("linear", "prepared", "step", "forward"):
        s["c_out"] = _f32(M, c["N"])
    if kind in ("prepared", "step"):
        s["a_prep"] = _bytes(cf.curvefp_prepared_bytes(M, K))
        s["ws"] = _bytes(cf.curvefp_gemm_prepared_workspace_bytes(M, c["N"], K))
    if kind == "prepared":
        s["w_prep"] = cf.curvefp_quantize_prepare(w, fmt, block=G)[2]
    if kind == "step":
        N = c["N"]
        s["w"], s["dst"] = w, _f32(M, K)
        s["out_w"] = (_codes(fmt, N, K), _scales(N, K // G), _bytes(cf.curvefp_prepared_bytes(N, K)))
    if kind == "forward":
        N = c["N"]
        s["w"], s["out_w"] = w, (_codes(fmt, N, K), _scales(N, K // G))
        s["ws"] = _bytes(cf.curvefp_gemm_workspace_bytes(M, N, K))
    return s


def run(s):
    c, x = s["c"], s["x"]
    kind, fmt, G, M, K = c["kind"], c["fmt"], c["block"], c["M"], c["K"]
    if kind == "backward":
        N = c["N"]
        q, qs = cf.curvefp_quantize(x, fmt, block=G, codes=s["codes"], scales=s["scales"])
        w, wsc = s["w_codes"]
        a, asc = s["x_codes"]
        # dX[M][K] = Q(dY)[M][N] . (W codes [N][K], read transposed)
        dx = cf.curvefp_gemm_mixed(q, qs, fmt, 0, w, wsc, c["fmt_b"], 1, M, K, N, block=G, c=s["dx"],
                                   workspace=s["ws"])
        # dW[N][K] = Q(dY)^T . X, both read transposed, contracted over the tokens
        dw = cf.curvefp_gemm_mixed(q, qs, fmt, 1, a, asc, c["fmt_b"], 1, N, K, M, block=G, c=s["dw"],
                                   workspace=s["ws"])
        return dict(codes=q, scales=qs, dx=dx, dw=dw)
    if kind == "tensorwise":
        q, qs = cf.curvefp_quantize_tensorwise(x, fmt, codes=s["codes"], scales=s["scales"], workspace=s["ws"])
        return dict(codes=q, scales=qs)
    if kind == "mse":
        q, qs = cf.curvefp_quantize_mse(x, fmt, candidates=c["candidates"], block=G, codes=s["codes"],
                                        scales=s["scales"])
        return dict(codes=q, scales=qs)
    if kind == "compact":
        q, ref, off = cf.curvefp_quantize_compact(x, fmt, G, c["bits"], codes=s["codes"], row_ref=s["ref"],
                                                  offsets=s["offsets"])
        qs = cf.curvefp_scales_unpack(ref, off, K // G, c["bits"], scales=s["scales"])
        y = cf.curvefp_dequantize(q, qs, fmt, M, K, block=G, dst=s["dst"])
        return dict(codes=q, ref=ref, offsets=off, scales=qs, y=y)
    if kind == "roundtrip":
        q, qs = cf.curvefp_quantize(x, fmt, block=G, codes=s["codes"], scales=s["scales"])
        y = cf.curvefp_dequantize(q, qs, fmt, M, K, block=G, dst=s["dst"])
        return dict(codes=q, scales=qs, y=y)
    N = c["N"]
    if kind == "prepared":
        q, qs, p = cf.curvefp_quantize_prepare(x, fmt, block=G, codes=s["codes"], scales=s["scales"],
                                               prepared=s["a_prep"])
        y = cf.curvefp_gemm_prepared(p, fmt, s["w_prep"], fmt, M, N, K, c=s["c_out"], workspace=s["ws"])
        return dict(codes=q, scales=qs, c=y)
    if kind == "step":
        (q, qs, p, d), (wq, wqs, wp) = cf.curvefp_quantize_prepare_pair(
            x, s["w"], fmt, block=G, out_a=(s["codes"], s["scales"], s["a_prep"], s["dst"]), out_b=s["out_w"])
        y = cf.curvefp_gemm_prepared(p, fmt, wp, fmt, M, N, K, c=s["c_out"], workspace=s["ws"])
        return dict(codes=q, scales=qs, w_codes=wq, w_scales=wqs, y=d, c=y)
    q, qs = cf.curvefp_quantize(x, fmt, block=G, codes=s["codes"], scales=s["scales"])
    if kind == "requant":
        w, wsc = s["w_codes"]
        oq, oqs = cf.curvefp_gemm_requant(q, qs, w, wsc, M, N, K, fmt, c["out_fmt"], block=G, out_codes=s["out"][0],
                                          out_scales=s["out"][1], workspace=s["ws"], out_block=c["out_block"])
        return dict(codes=q, scales=qs, out_codes=oq, out_scales=oqs)
    if kind == "forward":
        w, wsc = cf.curvefp_quantize(s["w"], fmt, block_axis=0, block=G, codes=s["out_w"][0], scales=s["out_w"][1])
        y = cf.curvefp_gemm_ws(q, qs, w, wsc, M, N, K, fmt, block=G, c=s["c_out"], workspace=s["ws"])
        return dict(codes=q, scales=qs, w_codes=w, w_scales=wsc, c=y)
    w, wsc = s["w_codes"]
    y = cf.curvefp_gemm_ws(q, qs, w, wsc, M, N, K, fmt, block=G, c=s["c_out"], workspace=s["ws"])
    return dict(codes=q, scales=qs, c=y)


# ---------------------------------------------------------------- work and tolerances

def work(case):
    """Bytes: the pass's tensors read once, its results written once, kept weights read once in the
    form they are kept as codes (expanded operands are this implementation's choice, not counted)."""
    c = case
    kind, fmt, G, M, K = c["kind"], c["fmt"], c["block"], c["M"], c["K"]
    e = 4 if c["dtype"] == "f32" else 2

    def q(rows, cols, f=fmt):                  # codes and scales of a tensor
        return _code_bytes(f, rows * cols) + rows * cols / G

    if kind == "backward":
        N, fb = c["N"], c["fmt_b"]
        return {"bytes": M * N * e + q(M, N) + q(M, K, fb) + q(N, K, fb) + 4.0 * (M * K + N * K),
                "flops": 4.0 * M * N * K}
    if kind in ("mse", "tensorwise"):
        scales = M if kind == "tensorwise" else M * K / G
        return {"bytes": M * K * e + _code_bytes(fmt, M * K) + scales, "flops": 0.0}
    if kind == "roundtrip":
        return {"bytes": M * K * (e + 4.0) + q(M, K), "flops": 0.0}
    if kind == "compact":
        nb = M * K / G
        return {"bytes": M * K * (e + 4.0) + _code_bytes(fmt, M * K) + M + nb * c["bits"] / 8 + nb, "flops": 0.0}
    N = c["N"]
    b = M * K * e + q(M, K) + q(N, K)
    if kind in ("step", "forward"):            # the weight's source belongs to the pass
        b += N * K * e
    if kind == "step":                         # the activation's reconstruction
        b += 4.0 * M * K
    if kind == "requant":
        b += _code_bytes(c["out_fmt"], M * N) + M * N / c["out_block"]
    else:
        b += 4.0 * M * N
    return {"bytes": b, "flops": 2.0 * M * N * K}


def tolerance(case):
    """Codes, scales and reconstructions have one right value.  A product is a sum of up to 14336
    fp32 terms: 2e-7 to 1.2e-6 from the exact sum in the 2-norm as measured against `exact`, and the
    order of the sum moves it by as much; four times the largest is allowed.  A requantized product
    moves a code only where a sum lies within that of a decision point (levels lie 9% apart: 1e-5 to
    5e-5 of the codes)."""
    if case["kind"] in ("mse", "compact", "roundtrip", "tensorwise"):
        return "exact"
    if case["kind"] == "requant":
        return {"rel": 0.0, "differ": 2e-4}
    return {"rel": 5e-6, "max": 1e-4}


# ---------------------------------------------------------------- 64-bit reference

def _levels(fmt):
    C, nmax, p, q = _FMT[fmt]
    n = torch.arange(-nmax, nmax + 1, dtype=torch.float64, device=_device())
    return torch.exp2(n * (p / float(q * 2 ** C)))


def _round_blocks(x, fmt, G, per_block=None):
    """Reconstruction in 64 bits of x quantized in blocks of G along its rows."""
    lev = _levels(fmt)
    top = float(lev[-1].to(torch.float32))
    bounds = torch.cat([lev[:1] / 2, (lev[1:] + lev[:-1]) / 2])
    values = torch.cat([torch.zeros_like(lev[:1]), lev])
    out = torch.empty(x.shape, dtype=torch.float64, device=x.device)
    step = max(1, (1 << 25) // x.shape[1])
    for r in range(0, x.shape[0], step):
        v = x[r:r + step].to(torch.float64)
        b = v.reshape(v.shape[0], -1, G)
        m, ex = torch.frexp(b.abs().amax(dim=2, keepdim=True) / top)   # amax / top = m 2^ex, m in [0.5, 1)
        a = torch.where(m == 0.5, ex - 1, ex).clamp(-127, 127)
        if per_block is not None:
            a = per_block(a)
        s = torch.exp2(a.to(torch.float64))
        y = b / s
        mag = values[torch.bucketize(y.abs(), bounds, right=True)]     # a tie goes to the level above
        out[r:r + step] = (torch.copysign(mag, y) * s).reshape(v.shape)
    return out


def _matmul(a, b):
    """a . b^T in 64 bits, in slices of rows."""
    out = torch.empty((a.shape[0], b.shape[0]), dtype=torch.float64, device=a.device)
    for r in range(0, a.shape[0], 2048):
        out[r:r + 2048] = torch.matmul(a[r:r + 2048], b.t())
    return out


def exact(case, seed):
    c = case
    kind, fmt, G, M, K = c["kind"], c["fmt"], c["block"], c["M"], c["K"]
    if kind in ("mse", "requant", "tensorwise"):
        return None
    if _device() == "cpu" and work(case)["flops"] > 2e11:
        return None
    x, w = _sources(c, seed)
    if kind == "roundtrip":
        return dict(codes=None, scales=None, y=_round_blocks(x, fmt, G))
    if kind == "compact":
        cap = 2 ** c["bits"] - 2

        def raised(a):                          # blocks far below their row's top take a raised scale
            return torch.maximum(a, a.amax(dim=1, keepdim=True) - cap)

        return dict(codes=None, ref=None, offsets=None, scales=None, y=_round_blocks(x, fmt, G, raised))
    if kind == "backward":
        xf, wf = w
        dy = _round_blocks(x, fmt, G)
        xq = _round_blocks(xf, c["fmt_b"], G)                          # [M][K]
        wq = _round_blocks(wf.t().contiguous(), c["fmt_b"], G)         # [N][K]
        return dict(codes=None, scales=None, dx=_matmul(dy, wq.t().contiguous()),
                    dw=_matmul(dy.t().contiguous(), xq.t().contiguous()))
    if kind == "forward":
        w = w.t().contiguous()
    xq, wq = _round_blocks(x, fmt, G), _round_blocks(w, fmt, G)
    y = _matmul(xq, wq)
    if kind == "step":
        return dict(codes=None, scales=None, w_codes=None, w_scales=None, y=xq, c=y)
    return dict(codes=None, scales=None, c=y)

"""The work that users of this library have it do, as cases that can be timed.

A case is a dict of plain values.  ``prepare`` makes what a program holds before the call (inputs, packed
weights, buffers, marshalled calls), ``run`` is one pass through the public entry points of
``paper_2307_15517_amd.mx``, ``work`` the bytes and operations a pass cannot do without and ``tolerance`` how far
two correct implementations of it may differ.

The kinds:

* ``decode``     the linear layers of one decoder layer (H->H, H->F, F->H) on 1..8 tokens: ``mx_linear``, fp32
                 activations in, weights packed once in the fragment layout.  A serving loop keeps its buffers, so the
                 calls are marshalled once (``mx.bound``).
* ``tokens``     the same packed weights on more tokens than ``mx_linear`` takes (a batch of sequences in decode, a
                 short prompt): ``mx_quantize_pack`` + ``mx_gemm`` on the fragment layout, exact block sums.
* ``prefill``    the same linears on a prompt, weights in the matrix layout: ``mx_quantize_pack`` + ``mx_gemm``.
* ``mlp``        a feed-forward pair whose hidden activations stay MXInt: ``mx_quantize_pack``, ``mx_gemm_q`` with an
                 MXInt bias (hidden activations never in fp32), ``mx_gemm`` back to fp32 for the residual sum.
* ``attention``  mixed-precision attention.  From fp32 Q, K and V (``cached`` false: a prompt), or fp32 Q against keys
                 and values that the program holds packed (``cached`` true: decoding, and chunks of a prompt).
* ``emulate``    what a search over formats does with a tensor: quantize, cast to a narrower width, dequantize,
                 results allocated by the convenience functions.
* ``minifloat``  the same for the Block Minifloat and Block Logarithm formats: quantize, dequantize.
"""
import math

import torch

from paper_2307_15517_amd import mx

FRAG, MAT = mx.MX_LAYOUT_FRAGMENT, mx.MX_LAYOUT_MATRIX
DEV = "cuda"


def listed():
    return [
        # one 768x768 linear on 16 tokens, the smallest call: launches and latency count
        dict(name="tokens_16x768", kind="tokens", M=16, H=768, F=0, block=16, wx=8, ww=4),
        # LLaMA-13B linears, one sequence decoding
        dict(name="decode_13b_m1", kind="decode", M=1, H=5120, F=13824, block=16, wx=8, ww=4),
        # LLaMA-13B linears, eight sequences decoding
        dict(name="decode_13b_m8", kind="decode", M=8, H=5120, F=13824, block=16, wx=8, ww=4),
        # LLaMA-7B sizes on five tokens, blocks of 32 and widths as a mixed-precision search hands them out
        dict(name="decode_7b_m5_w65", kind="decode", M=5, H=4096, F=11008, block=32, wx=6, ww=5),
        # LLaMA-13B linears, a batch of 32 sequences on the weights packed for decoding
        dict(name="tokens_13b_m32", kind="tokens", M=32, H=5120, F=13824, block=16, wx=8, ww=4),
        # OPT-125M linears on a sequence of 128
        dict(name="prefill_opt125m_128", kind="prefill", M=128, H=768, F=3072, block=16, wx=6, ww=4),
        # LLaMA-7B linears on a prompt of 2048: the largest
        dict(name="prefill_7b_2048", kind="prefill", M=2048, H=4096, F=11008, block=32, wx=8, ww=4),
        # a feed-forward pair of LLaMA-7B size on a prompt of odd length, hidden activations MXInt
        dict(name="mlp_7b_333", kind="mlp", M=333, H=4096, F=11008, block=32, wx=8, ww=4),
        # attention of a 2048-token prompt, widths drawn per tensor
        dict(name="attn_32x2048x128", kind="attention", heads=32, Sq=2048, Sk=2048, D=128, wq=7, wk=6, wp=5, wv=3,
             bp=16, rp=1, cached=False),
        # one new token of one sequence against 1936 cached positions
        dict(name="attn_decode_1936", kind="attention", heads=32, Sq=1, Sk=1936, D=128, wq=8, wk=8, wp=8, wv=8,
             bp=16, rp=1, cached=True),
        # a LLaMA-7B activation tensor through the quantizer, a cast and back
        dict(name="emulate_2048x11008", kind="emulate", rows=2048, cols=11008, block=32, w=8, w2=5, rows2=1),
        # a LLaMA-7B weight tensor's share in Block Minifloat, odd number of rows
        dict(name="minifloat_1001x4096", kind="minifloat", rows=1001, cols=4096, block=16, e=4, m=3),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _mult(v, m, lo):
    return max(lo, int(v) // m * m)


def draw(rng):
    kind = rng.choice(["decode", "decode", "tokens", "tokens", "prefill", "prefill", "mlp", "attention", "attention",
                       "emulate", "minifloat"])
    if kind in ("decode", "tokens", "prefill", "mlp"):
        block = rng.choice([16, 32])
        M = {"decode": lambda: rng.randint(1, 8), "tokens": lambda: int(_log(rng, 9, 129)),
             "prefill": lambda: int(_log(rng, 16, 2048.99)), "mlp": lambda: int(_log(rng, 16, 2048.99))}[kind]()
        H = _mult(_log(rng, 768, 5120 if M <= 128 else 4096), block, block)
        F = _mult(min(H * rng.uniform(2.0, 4.0), 13824 if M <= 128 else 11008), block, block)
        wide = kind in ("decode", "tokens")
        return dict(kind=kind, M=M, H=H, F=F, block=block, wx=rng.randint(5, 8),
                    ww=rng.choice([3, 4, 4, 4, 5, 6, 8] if wide else [2, 3, 4, 4, 4]))
    if kind == "attention":
        cached = rng.random() < 0.5
        Sk = _mult(_log(rng, 64, 2048.99), 32, 32)
        Sq = int(_log(rng, 1, min(512, Sk))) if cached else Sk - rng.randint(0, 31)
        return dict(kind=kind, heads=rng.randint(8, 32), Sq=Sq, Sk=Sk, D=rng.choice([64, 80, 96, 128]),
                    wq=rng.randint(4, 8), wk=rng.randint(4, 8), wp=rng.randint(3, 8), wv=rng.randint(3, 8),
                    bp=rng.choice([16, 32]), rp=2 if Sq % 2 == 0 and rng.random() < 0.3 else 1, cached=cached)
    if kind == "emulate":
        block = rng.choice([16, 32, 64])
        w = rng.randint(4, 8)
        rows2 = rng.choice([1, 1, 2])
        return dict(kind=kind, rows=_mult(_log(rng, 16, 2048.99), rows2, 2), cols=_mult(_log(rng, 768, 11008), block, block),
                    block=block, w=w, w2=rng.randint(2, w), rows2=rows2)
    e = rng.randint(2, 7)
    block = rng.choice([16, 32])
    return dict(kind=kind, rows=int(_log(rng, 16, 2048.99)), cols=_mult(_log(rng, 768, 11008), block, block), block=block,
                e=e, m=rng.randint(0, 7 - e))


# ---- inputs -----------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _activations(g, *shape):
    """Heavy-tailed activations with outlier channels: Student-t with three degrees of freedom, 1 % of the
    channels (at least one) scaled by 100."""
    x = torch.randn(shape, generator=g, device=DEV)
    chi = sum(torch.randn(shape, generator=g, device=DEV).square_() for _ in range(3))
    x /= chi.div_(3.0).sqrt_().clamp_(min=1e-3)
    cols = shape[-1]
    ch = torch.randperm(cols, generator=g, device=DEV)[:max(1, round(0.01 * cols))]
    x[..., ch] *= 100.0
    return x


def _heads(g, heads, n, dim):
    """One of Q, K, V: N(0, 1), 1 % of the channels (at least one) scaled by 50."""
    x = torch.randn((heads, n, dim), generator=g, device=DEV)
    ch = torch.randperm(dim, generator=g, device=DEV)[:max(1, round(0.01 * dim))]
    x[..., ch] *= 50.0
    return x


def _weights(g, n, k, f, layout):
    return mx.quantize_pack(torch.randn((n, k), generator=g, device=DEV) * 0.02, f, layout)


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device=DEV)


def _linears(case):
    """(K, N) of the case's linear layers."""
    H, F = case["H"], case["F"]
    return [(H, H), (H, F), (F, H)] if F else [(H, H)]


# ---- prepare and run ----------------------------------------------------------------------------------
def prepare(case, seed):
    return {"decode": _prepare_decode, "tokens": _prepare_linears, "prefill": _prepare_linears, "mlp": _prepare_mlp,
            "attention": _prepare_attention, "emulate": _prepare_tensor,
            "minifloat": _prepare_tensor}[case["kind"]](case, _gen(seed))


def _prepare_decode(case, g):
    M, fx, fw = case["M"], mx.fmt(case["block"], case["wx"]), mx.fmt(case["block"], case["ww"])
    s = dict(case=case, calls=[], keep=[], out=[])
    need = max(mx.mx_linear_workspace_bytes(M, K, N, fx, fw) for K, N in _linears(case))
    ws = torch.zeros(need, dtype=torch.uint8, device=DEV)         # one workspace serves call after call
    for K, N in _linears(case):
        x, w = _activations(g, M, K), _weights(g, N, K, fw, FRAG)
        y = torch.empty((M, N), dtype=torch.float32, device=DEV)
        s["calls"].append(mx.bound("mx_linear", x, M, K, K, fx, ws, w, N, fw, FRAG, y, N))
        s["keep"] += [x, w, ws]
        s["out"].append(y)
    return s


def _prepare_linears(case, g):
    layout = FRAG if case["kind"] == "tokens" else MAT
    M, fx, fw = case["M"], mx.fmt(case["block"], case["wx"]), mx.fmt(case["block"], case["ww"])
    s = dict(case=case, calls=[], keep=[], out=[])
    for K, N in _linears(case):
        x, w = _activations(g, M, K), _weights(g, N, K, fw, layout)
        p = _bytes(mx.mx_packed_bytes(1, M, K, fx, layout))
        y = torch.empty((M, N), dtype=torch.float32, device=DEV)
        s["calls"].append(mx.bound("mx_quantize_pack", x, 1, M, K, K, 0, fx, layout, p))
        s["calls"].append(mx.bound("mx_gemm", 1, M, N, K, p, fx, w, fw, layout, y, N, 0))
        s["keep"] += [x, w, p]
        s["out"].append(y)
    return s


def _prepare_mlp(case, g):
    M, H, F = case["M"], case["H"], case["F"]
    fx, fw = mx.fmt(case["block"], case["wx"]), mx.fmt(case["block"], case["ww"])
    return dict(case=case, fx=fx, fw=fw, x=_activations(g, M, H), xp=_bytes(mx.mx_packed_bytes(1, M, H, fx, MAT)),
                w1=_weights(g, F, H, fw, MAT), w2=_weights(g, H, F, fw, MAT),
                bias=mx.quantize(torch.randn((1, F), generator=g, device=DEV), fw),
                hp=_bytes(mx.mx_packed_bytes(1, M, F, fx, MAT)),
                y=torch.empty((M, H), dtype=torch.float32, device=DEV))


def _prepare_attention(case, g):
    h, Sq, Sk, D = case["heads"], case["Sq"], case["Sk"], case["D"]
    s = dict(case=case, fq=mx.fmt(16, case["wq"]), fk=mx.fmt(16, case["wk"]), fv=mx.fmt(16, case["wv"]),
             fp=mx.fmt(case["bp"], case["wp"], block_rows=case["rp"]), q=_heads(g, h, Sq, D), k=_heads(g, h, Sk, D),
             v=_heads(g, h, Sk, D))
    s["qp"] = _bytes(mx.mx_packed_bytes(h, Sq, D, s["fq"], MAT))
    s["kp"] = _bytes(mx.mx_packed_bytes(h, Sk, D, s["fk"], MAT))
    s["vp"] = _bytes(mx.mx_packed_bytes(h, D, Sk, s["fv"], MAT))
    s["o"] = torch.empty((h, Sq, D), dtype=torch.float32, device=DEV)
    if case["cached"]:
        _pack_kv(s)
        del s["k"], s["v"]
    return s


def _prepare_tensor(case, g):
    return dict(case=case, x=_activations(g, case["rows"], case["cols"]))


def _pack_kv(s):
    c = s["case"]
    h, Sk, D = c["heads"], c["Sk"], c["D"]
    mx.mx_quantize_pack(s["k"], h, Sk, D, D, Sk * D, s["fk"], MAT, s["kp"])
    mx.mx_quantize_pack_axis0(s["v"], h, Sk, D, D, Sk * D, s["fv"], MAT, s["vp"])


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind in ("decode", "tokens", "prefill"):
        for call in state["calls"]:
            call()
        return state["out"]
    if kind == "mlp":
        s, M, H, F = state, c["M"], c["H"], c["F"]
        mx.mx_quantize_pack(s["x"], 1, M, H, H, 0, s["fx"], MAT, s["xp"])
        mx.mx_gemm_q(1, M, F, H, s["xp"], s["fx"], s["w1"], s["fw"], MAT, *s["bias"], s["fw"], s["fx"], s["hp"])
        mx.mx_gemm(1, M, H, F, s["hp"], s["fx"], s["w2"], s["fw"], MAT, s["y"], H, 0)
        return s["y"]
    if kind == "attention":
        s, h, Sq, Sk, D = state, c["heads"], c["Sq"], c["Sk"], c["D"]
        mx.mx_quantize_pack(s["q"], h, Sq, D, D, Sq * D, s["fq"], MAT, s["qp"])
        if not c["cached"]:
            _pack_kv(s)
        mx.mx_attention(h, Sq, Sk, D, s["qp"], s["fq"], s["kp"], s["fk"], s["vp"], s["fv"], s["fp"], D ** -0.5, MAT,
                        s["o"], D, Sq * D)
        return s["o"]
    if kind == "emulate":
        rows, cols = c["rows"], c["cols"]
        f8, f2 = (mx.fmt(c["block"], w, block_rows=c["rows2"]) for w in (c["w"], c["w2"]))
        mant, exps = mx.quantize(state["x"], f8)
        mant2, exps2 = mx.cast(mant, exps, 1, rows, cols, f8, f2)
        return mant, exps, mant2, exps2, mx.dequantize(mant2, exps2, 1, rows, cols, f2)
    rows, cols = c["rows"], c["cols"]
    f = mx.mx_minifloat_format(c["block"], c["e"], c["m"], mx.MX_RNE)
    codes, shared = _bytes(rows * cols), _bytes(rows * cols // c["block"])
    mx.mx_quantize_minifloat(state["x"], 1, rows, cols, cols, 0, f, codes, shared)
    y = torch.empty((rows, cols), dtype=torch.float32, device=DEV)
    mx.mx_dequantize_minifloat(codes, shared, 1, rows, cols, f, y)
    return codes, shared, y


# ---- what a pass cannot do without, and how exact it is -------------------------------------------------
def _density(w, block):
    return w / 8.0 + 1.0 / block


def work(case):
    kind = case["kind"]
    if kind in ("decode", "tokens", "prefill"):
        M, dw = case["M"], _density(case["ww"], case["block"])
        return {"bytes": sum(4.0 * M * K + dw * N * K + 4.0 * M * N for K, N in _linears(case)),
                "flops": sum(2.0 * M * N * K for K, N in _linears(case))}
    if kind == "mlp":
        M, H, F = case["M"], case["H"], case["F"]
        return {"bytes": 8.0 * M * H + 2 * _density(case["ww"], case["block"]) * H * F, "flops": 4.0 * M * H * F}
    if kind == "attention":
        h, Sq, Sk, D = case["heads"], case["Sq"], case["Sk"], case["D"]
        kv = _density(case["wk"], 16) + _density(case["wv"], 16) if case["cached"] else 8.0
        return {"bytes": h * D * (8.0 * Sq + kv * Sk), "flops": 4.0 * h * Sq * Sk * D}
    n = float(case["rows"] * case["cols"])
    if kind == "emulate":
        b = case["block"] * case["rows2"]
        return {"bytes": n * (8.0 + _density(case["w"], b) + _density(case["w2"], b)), "flops": 0.0}
    return {"bytes": n * (8.0 + _density(8, case["block"])), "flops": 0.0}


def tolerance(case):
    kind = case["kind"]
    # Against the same path in float64 (dequantized operands) the products differ by at most 2e-8 in the 2-norm and
    # 1.2e-7 at the worst element (most are exact), attention by 2.3e-3 and 0.084: a probability within a few 1e-6 of a
    # tie of its quantizer takes the neighbouring mantissa, a block maximum that close to a power of two the
    # neighbouring exponent.
    if kind in ("decode", "tokens", "prefill"):
        return {"rel": 1e-6, "max": 1e-5}                 # block sums exact, fp32 sums over the blocks
    if kind == "mlp":
        return {"rel": 2e-5, "max": 2e-3}                 # a hidden value at a tie moves a sum by a step of one operand
    if kind == "attention":
        return {"rel": 8e-3, "max": 0.35}
    return "exact"

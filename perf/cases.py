"""The work this library is measured by: calls of its public entry points as a user's program
makes them, over the range of shapes, operand types and chains such programs have.

A case is a dict of plain values:

    kind    "fused": fused_gemm_epilogue, "gated": fused_gated_gemm_epilogue, "rows": fge_row_op
    dtype   of X and W ("rows": of the matrix): f32, bf16, f16, f8 (E4M3);   out: of the result
    batch   problems of M rows that share W (1: a plain matrix)
    M, K, N rows, contraction length, columns ("rows": K is 0)
    act, norm   names of the activation and of the row operation
    bias, gamma, beta   whether the vector is given
    alpha, post         result = rowop(act(post * (alpha * X.W^T + b)))

`listed()` holds one case per kind of use, at the size its users know best; `draw()` gives
others of the same uses over the whole range of sizes, with rows, columns and contraction lengths
off every tile boundary and, more rarely, off the 16-byte grid."""
import math

import torch

from paper_2512_23424_amd import binding as fge

DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "f8": torch.float8_e4m3fn}
BYTES = {"f32": 4, "bf16": 2, "f16": 2, "f8": 1}
EPS = {"layernorm": 1e-5, "rmsnorm": 1e-6}


def _case(kind, dtype, out, M, K, N, act, norm, batch=1, bias=False, gamma=False, beta=False, alpha=1.0, post=1.0):
    return {"kind": kind, "dtype": dtype, "out": out, "batch": batch, "M": M, "K": K, "N": N, "act": act, "norm": norm,
            "bias": bias, "gamma": gamma, "beta": beta, "alpha": alpha, "post": post}


def listed():
    """One case per use."""
    cases = {
        # a tiny fp32 head (a router, a small classifier): one launch, the call's latency
        "head_f32": _case("fused", "f32", "f32", 64, 64, 64, "relu", "softmax", bias=True),
        # a dense layer in fp32 with its normalisation
        "dense_f32": _case("fused", "f32", "f32", 4096, 1024, 1024, "gelu_tanh", "layernorm", bias=True, gamma=True, beta=True),
        # the projection of a large bf16 model over a full training or prefill batch
        "projection_bf16": _case("fused", "bf16", "bf16", 8192, 4096, 4096, "silu", "rmsnorm", gamma=True),
        # a batch of problems with a short contraction and one set of weights (scores, then softmax)
        "scores_bf16": _case("fused", "bf16", "bf16", 2048, 512, 2048, "gelu_erf", "softmax", batch=16, bias=True,
                             alpha=1 / math.sqrt(512)),
        # very many short rows through a narrow layer: output bound, values and logsumexp returned
        "narrow_f32": _case("fused", "f32", "f32", 262144, 64, 512, "clamp", "logsumexp", bias=True, post=2.0),
        # the projection with 8-bit operands and a per-tensor scale
        "projection_f8": _case("fused", "f8", "bf16", 8192, 4096, 4096, "silu", "rmsnorm", gamma=True, alpha=1 / 64),
        # the gated feed-forward of a large bf16 model
        "gated_bf16": _case("gated", "bf16", "bf16", 8192, 4096, 4096, "silu", "rmsnorm", gamma=True),
        # one decode step of a small batch: every weight read for a few rows
        "decode_bf16": _case("fused", "bf16", "bf16", 16, 4096, 4096, "silu", "rmsnorm", gamma=True),
        # ... and of the gated layer
        "decode_gated_bf16": _case("gated", "bf16", "bf16", 16, 4096, 4096, "silu", "none"),
        # a prefill of an ordinary prompt: a row count of no particular shape
        "prefill_f16": _case("fused", "f16", "f16", 1000, 4096, 4096, "gelu_erf", "layernorm", bias=True, gamma=True, beta=True),
        # vocabulary logits with their logsumexp (a loss), the vocabulary being odd
        "logits_bf16": _case("fused", "bf16", "bf16", 2048, 4096, 50257, "none", "logsumexp", bias=True),
        # a normalisation on its own
        "rows_bf16": _case("rows", "bf16", "bf16", 65536, 0, 4096, "none", "rmsnorm", gamma=True),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _size(rng, lo, hi, grid, odd=0.0):
    """Spread over the logarithm of lo .. hi; a third powers of two, the rest multiples of `grid`
    (a share `odd` of all: any number)."""
    v = lo * (hi / lo) ** rng.random()
    r = rng.random()
    if r < odd:
        v = int(v)
    elif r < odd + (1 - odd) / 3:
        v = 2 ** round(math.log2(v))
    else:
        v = round(v / grid) * grid
    return max(lo, min(hi, v))


def draw(rng):
    """One more case of the same uses."""
    use = rng.choice(["head", "dense", "projection", "scores", "narrow", "projection_f8", "gated", "decode", "decode_gated",
                      "prefill", "logits", "rows"])
    acts = ["none", "relu", "gelu_tanh", "gelu_erf", "silu"]
    norms = ["none", "softmax", "layernorm", "rmsnorm", "logsumexp"]
    half = rng.choice(["bf16", "bf16", "f16"])
    act, norm = rng.choice(acts), rng.choice(norms)
    bias, affine = rng.random() < 0.5, rng.random() < 0.7
    norm = {"scores": rng.choice(["softmax", "softmax", norm]), "narrow": rng.choice(["logsumexp", norm]),
            "gated": rng.choice(["none", "rmsnorm", norm]), "decode_gated": rng.choice(["none", "none", "rmsnorm"]),
            "logits": rng.choice(["logsumexp", "softmax", "none"]), "rows": rng.choice(norms[1:])}.get(use, norm)
    kw = {"bias": bias, "gamma": affine and norm in ("layernorm", "rmsnorm"), "beta": affine and norm == "layernorm"}

    def within(M, K, N, limit, least=1):                 # fewer rows where the product would be too large
        return max(least, min(M, int(limit / (K * N))))

    if use == "head":
        return _case("fused", "f32", "f32", _size(rng, 1, 512, 1), _size(rng, 16, 512, 4, 0.3), _size(rng, 16, 512, 4, 0.3), act, norm, **kw)
    if use == "dense":
        K, N = _size(rng, 128, 4096, 4, 0.15), _size(rng, 128, 4096, 4, 0.15)
        M = within(_size(rng, 512, 16384, 1), K, N, 2.0 ** 35)
        return _case("fused", "f32", rng.choice(["f32", "f32", "bf16"]), M, K, N, act, norm, **kw)
    if use in ("projection", "prefill"):
        K, N = _size(rng, 512, 8192, 8, 0.1), _size(rng, 512, 8192, 8, 0.1)
        M = within(_size(rng, 65, 2048, 1) if use == "prefill" else _size(rng, 2048, 16384, 1), K, N, 2.0 ** 37)
        return _case("fused", half, rng.choice([half, half, half, "f32"]), M, K, N, act, norm, **kw)
    if use == "scores":
        K, N, B = _size(rng, 64, 1024, 8), _size(rng, 128, 4096, 8), rng.randint(2, 32)
        M = within(_size(rng, 64, 4096, 1), K * B, N, 2.0 ** 35)
        return _case("fused", half, half, M, K, N, act, norm, batch=B, alpha=1 / math.sqrt(K), **kw)
    if use == "narrow":
        K, N = _size(rng, 16, 64, 4), _size(rng, 64, 512, 4)
        M = within(_size(rng, 4096, 1 << 19, 1), 1, N, 2.0 ** 27)
        return _case("fused", "f32", "f32", M, K, N, rng.choice(acts + ["clamp"]), norm, post=2.0, **kw)
    if use == "projection_f8":
        K, N = _size(rng, 512, 8192, 16), _size(rng, 512, 8192, 16)
        M = within(_size(rng, 256, 16384, 1), K, N, 2.0 ** 37)
        return _case("fused", "f8", "bf16", M, K, N, act, norm, alpha=1 / math.sqrt(K), **kw)
    if use == "gated":
        K, N = _size(rng, 512, 8192, 8), _size(rng, 512, 11008, 8)
        M = within(_size(rng, 128, 8192, 1), K, N, 2.0 ** 37)
        return _case("gated", half, half, M, K, N, rng.choice(["silu", "silu", "gelu_erf", "gelu_tanh"]), norm, **kw)
    if use == "decode":
        t = rng.choice([half, half, "f8"])
        return _case("fused", t, half if t != "f8" else "bf16", _size(rng, 1, 64, 1), _size(rng, 1024, 8192, 16), _size(rng, 1024, 8192, 16), act, norm,
                     alpha=1 / 64 if t == "f8" else 1.0, **kw)
    if use == "decode_gated":
        return _case("gated", half, half, _size(rng, 1, 64, 1), _size(rng, 1024, 8192, 8), _size(rng, 1024, 11008, 8),
                     rng.choice(["silu", "silu", "gelu_erf", "gelu_tanh"]), norm, **kw)
    if use == "logits":
        K, N = _size(rng, 1024, 4096, 8), rng.choice([32000, 50257, 32768, rng.randint(16384, 50257)])
        return _case("fused", half, half, _size(rng, 16, 2048, 1), K, N, "none", norm, **kw)
    N = _size(rng, 256, 32000, 8, 0.1)
    t = rng.choice(["bf16", "f16", "f32"])
    return _case("rows", t, t, within(_size(rng, 16, 1 << 18, 1), 1, N, 2.0 ** 28), 0, N, "none", norm, **dict(kw, bias=False))


def prepare(case, seed):
    """Operands, the parameter struct and the workspace, as a program holds them before the call."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, M, K, N = case["batch"], case["M"], case["K"], case["N"]

    def normal(*shape, std=1.0):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32) * std

    def uniform(*shape, lo, hi):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float32) * (hi - lo) + lo

    dt, od = DTYPE[case["dtype"]], DTYPE[case["out"]]
    lead = (B,) if B > 1 else ()
    out = torch.empty(*lead, M, N, device="cuda", dtype=od)
    s = {"case": case, "out": out, "X": None, "W": None, "W2": None, "b": None, "b2": None}
    s["gamma"] = 1 + normal(N, std=0.1) if case["gamma"] else None
    s["beta"] = normal(N, std=0.1) if case["beta"] else None
    s["aux"] = torch.empty(B * M, device="cuda", dtype=torch.float32) if case["norm"] == "logsumexp" else None
    common = {"eps": EPS.get(case["norm"], 0.0), "gamma": s["gamma"], "beta": s["beta"], "aux_out": s["aux"]}
    if case["kind"] == "rows":
        s["X"] = normal(M, N, std=2.0).to(dt)
        s["p"] = fge.make_params(None, None, out, **common)
        return s
    s["X"] = normal(*lead, M, K).to(dt)
    # unit-variance results; 8-bit weights keep unit variance themselves, alpha scales the product
    std = 1.0 if case["dtype"] == "f8" else 1.0 / math.sqrt(K)
    s["W"] = normal(N, K, std=std).to(dt)
    s["b"] = uniform(N, lo=-0.1, hi=0.1) if case["bias"] else None
    common.update(alpha=case["alpha"], post_scale=case["post"], clamp_lo=-5.0, clamp_hi=5.0)
    p = s["p"] = fge.make_params(s["X"], s["W"], out, **common)
    if case["kind"] == "gated":
        s["W2"] = normal(N, K, std=std).to(dt)
        s["b2"] = uniform(N, lo=-0.1, hi=0.1) if case["bias"] else None
        n = fge.fge_gated_workspace_bytes(True, case["act"], case["norm"], p)
    else:
        n = fge.fge_workspace_bytes(True, case["act"], case["norm"], p)
    s["ws"] = torch.empty(max(n, 16), device="cuda", dtype=torch.uint8)
    p.workspace, p.workspace_bytes = s["ws"].data_ptr(), s["ws"].numel()
    return s


def run(s):
    """One call; the result, with the row logsumexp beside it where the chain has one."""
    c = s["case"]
    if c["kind"] == "rows":
        fge.fge_row_op(s["X"], c["norm"], s["p"], s["out"])
    elif c["kind"] == "gated":
        fge.fused_gated_gemm_epilogue(s["X"], s["W"], s["W2"], s["b"], s["b2"], c["act"], c["norm"], s["p"], s["out"])
    else:
        fge.fused_gemm_epilogue(s["X"], s["W"], s["b"], c["act"], c["norm"], s["p"], s["out"])
    return s["out"] if s["aux"] is None else (s["out"], s["aux"])


def work(case):
    """Operands and vectors read once, results written once; two operations per multiply-add and,
    for a row operation on its own, about four per value."""
    B, M, K, N = case["batch"], case["M"], case["K"], case["N"]
    rows = B * M
    vectors = 4 * N * (case["gamma"] + case["beta"])
    results = rows * N * BYTES[case["out"]] + (4 * rows if case["norm"] == "logsumexp" else 0)
    if case["kind"] == "rows":
        return {"bytes": rows * N * BYTES[case["dtype"]] + results + vectors, "flops": 4 * rows * N}
    products = 2 if case["kind"] == "gated" else 1
    operands = (rows * K + products * N * K) * BYTES[case["dtype"]]
    return {"bytes": operands + results + vectors + 4 * N * case["bias"] * products, "flops": 2 * products * rows * N * K}


def tolerance(case):
    """About four times what the path showed against float64 on the listed cases and thirty drawn
    ones.  16-bit results: one rounding (bf16 1.7e-3, f16 2.1e-4 in the 2-norm), a second one where
    a row is parked in the result's type before it is normalised (2.4e-3, 3.0e-4; largest 7.7e-3,
    1.0e-3; f16 probabilities of a wide softmax lie in its subnormal range: 5.2e-4, 1.3e-3).  fp32 results of bf16 / f16 operands: exact products, fp32 sums.  fp32 operands: split
    into two bf16 terms unless the IEEE flag is set (5e-6, largest 6e-5).  E4M3 operands: the
    64-term sums of the 8-bit matrix instruction (2.3e-4).  Row operations in fp32: 6e-8."""
    if case["out"] == "bf16":
        return {"rel": 8e-3, "max": 3e-2}
    if case["out"] == "f16":
        return {"rel": 2e-3, "max": 5e-3}
    if case["kind"] == "rows":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 2e-5, "max": 2.5e-4}

"""The work this framework is used for, as a list of measurable cases.

Four kinds of call, each through the package's public entry points:

  linear   one W4A4 (or W4A8) linear layer: transform + clip + quantise the activations, then the block-scaled GEMM
  mlp      a gated MLP block behind an RMSNorm: row factors, gate/up GEMM with the gated epilogue, down projection
  kv       one attention step's cache work for a key and a value cache: append the new tokens, read the context
           back as bf16, transform the queries (inverse transpose) and the attention output (inverse)
  convert  offline preparation of one weight matrix for a checkpoint: inverse transform, MXFP4, export

The shapes are the repository's own workloads (an 8B-class decoder with hidden size 4096 and intermediate size 14336,
a multimodal MLP with 3584 / 18944, a cache of 8 heads x 128 channels) from one token to 8192 tokens.
"""
import math

import numpy as np
import torch

import paper_2603_16590_amd as B

# the costliest listed case; a drawn case is scaled down to at most this
MOST_FLOPS = 2.0 * 8192 * 3584 * 18944


def listed():
    def linear(name, M, K, N, bits=4, x="bf16", y="bf16", dist="outliers"):
        return {"name": name, "op": "linear", "M": M, "K": K, "N": N, "bits": bits, "x": x, "y": y, "dist": dist}

    return [
        # a small layer in fp32: everything is launch and host time
        linear("linear-tiny-f32", 64, 256, 256, x="f32", y="f32"),
        # the query projection of a decode step with 16 sequences
        linear("linear-decode", 16, 4096, 4096),
        # the MLP block of a decode step for one user
        {"name": "mlp-decode", "op": "mlp", "M": 1, "D": 4096, "F": 14336, "bits": 4},
        # attention of a decode step over a context of 8192 tokens with an 8-bit cache
        {"name": "kv-decode", "op": "kv", "M": 1, "context": 8192, "C": 1024, "Q": 4096, "bits": 8},
        # a prefill chunk of odd length, widths that are no multiple of any tile
        linear("linear-ragged", 333, 3616, 5000, y="f32"),
        # the down projection of a chunk of 512 tokens (chunked prefill, large decode batches)
        linear("linear-chunk-down", 512, 14336, 4096, dist="heavy"),
        # prefill of an 8B-class model: up or gate projection, down projection
        linear("linear-prefill-up", 2048, 4096, 14336, dist="tokens"),
        linear("linear-prefill-down", 4096, 14336, 4096, dist="heavy"),
        # the same up projection with 8-bit activations (the near-lossless setting)
        linear("linear-prefill-a8", 2048, 4096, 14336, bits=8, dist="tokens"),
        # the whole MLP block of a prefill
        {"name": "mlp-prefill", "op": "mlp", "M": 2048, "D": 4096, "F": 14336, "bits": 4},
        # a multimodal prompt: image tokens followed by text tokens
        linear("linear-multimodal", 8192, 3584, 18944, dist="image"),
        # loading a checkpoint: one projection prepared and exported
        {"name": "convert-up", "op": "convert", "K": 4096, "N": 14336, "w": "bf16", "kxn": True},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, lo, hi, step):
    return max(lo, int(round(_log(rng, lo, hi) / step)) * step)


def draw(rng):
    op = rng.choice(["linear"] * 5 + ["mlp"] * 2 + ["kv", "convert"])
    M = int(round(_log(rng, 1, 8192)))
    bits = rng.choice([4, 4, 4, 8])
    if op == "linear":
        K, N = _width(rng, 256, 14336, 32), _width(rng, 64, 18944, rng.choice([1, 8, 64]))
        M = min(M, int(MOST_FLOPS / (2.0 * K * N * (1 if bits == 4 else 2))))
        return {"op": op, "M": M, "K": K, "N": N, "bits": bits, "x": rng.choice(["bf16"] * 6 + ["f32"]),
                "y": rng.choice(["bf16", "bf16", "f32"]), "dist": rng.choice(["outliers", "tokens", "heavy", "image"])}
    if op == "mlp":
        D, F = _width(rng, 1024, 4096, 32), _width(rng, 2048, 14336, 32)
        return {"op": op, "M": min(M, int(MOST_FLOPS / (6.0 * D * F * (1 if bits == 4 else 2)))), "D": D, "F": F, "bits": bits}
    if op == "kv":
        return {"op": op, "M": min(M, 2048), "context": int(round(_log(rng, 64, 32768))), "C": 128 * rng.randint(1, 16),
                "Q": 128 * rng.randint(8, 32), "bits": rng.choice([4, 8])}
    return {"op": op, "K": _width(rng, 256, 4096, 32), "N": _width(rng, 64, 14336, 1), "w": rng.choice(["bf16", "bf16", "f32"]),
            "kxn": rng.choice([True, False])}


_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _transform(rng, K, clip=True):
    """Global-and-private Kronecker factors near the identity and learned clip ratios."""
    G = (np.eye(4) + 0.05 * rng.standard_normal((4, 4))).astype(np.float32)
    P = (np.eye(8) + 0.05 * rng.standard_normal((K // 32, 8, 8))).astype(np.float32)
    ratio = rng.uniform(0.85, 1.0, K // 32).astype(np.float32) if clip else None
    return G, P, ratio


def _weight(gen, K, N):
    return (torch.randn((K, N), device="cuda", generator=gen) * 0.02).to(torch.bfloat16)


def _activations(gen, dist, M, K):
    """Activations as a language model's projections see them: outlier channels, uneven tokens, heavy tails."""
    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen)

    X = normal(M, K)
    if dist == "heavy":                                     # Student t with 3 degrees of freedom
        X *= torch.rsqrt((normal(M, K).square_() + normal(M, K).square_() + normal(M, K).square_()) / 3.0)
    elif dist == "tokens":
        X *= torch.exp(0.5 * normal(M, 1))
    chans = torch.randperm(K, device="cuda", generator=gen)[: max(1, K // 100)]
    if dist == "image":                                     # three quarters image tokens: two modes, no outliers
        cut = M - M // 4
        X[:cut] = 2.0 * X[:cut] + 1.5 * torch.sign(normal(cut, K))
        X[cut:, chans] *= 30.0
    else:
        X[:, chans] *= 50.0 if dist == "heavy" else 30.0
    return X


def _bytes(n):
    return torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    op = case["op"]
    s = {"op": op, "bits": case.get("bits", 4)}
    if op == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        s["t"] = B.Transform(K, *_transform(rng, K))
        s["w"] = B.batq_prepare_weight(s["t"], _weight(gen, K, N))
        s["X"] = _activations(gen, case["dist"], M, K).to(_DTYPE[case["x"]])
        s["Y"] = torch.empty((M, N), dtype=_DTYPE[case["y"]], device="cuda")
        s["ws"] = _bytes(B.batq_linear_workspace_for(s["w"], M, s["bits"]))
    elif op == "mlp":
        M, D, F = case["M"], case["D"], case["F"]
        G, P, clip = _transform(rng, D)
        # the norm weight is folded into the blocks: RMSNorm(x) T = r (x diag(gamma)) T
        gamma = (1.0 + 0.1 * rng.standard_normal(D)).astype(np.float32).reshape(D // 32, 32, 1)
        T = np.stack([np.kron(G, p) for p in P])
        s["t_in"] = B.Transform.general(D, dense=gamma * T, clip=clip)
        s["t_down"] = B.Transform(F, *_transform(rng, F))
        s["w_in"] = B.batq_prepare_weight_gate_up(B.Transform(D, G, P, clip), _weight(gen, D, F), _weight(gen, D, F))
        s["w_down"] = B.batq_prepare_weight(s["t_down"], _weight(gen, F, D))
        s["X"] = _activations(gen, "outliers", M, D).to(torch.bfloat16)
        s["H"] = torch.empty((M, F), dtype=torch.bfloat16, device="cuda")
        s["Y"] = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
        s["ws"] = _bytes(max(B.batq_linear_workspace_for(s["w_in"], M, s["bits"]),
                             B.batq_linear_workspace_for(s["w_down"], M, s["bits"])))
    elif op == "kv":
        M, L, C, Q = case["M"], case["context"], case["C"], case["Q"]
        s["L"], s["cap"] = L, -(-(L + M) // 256) * 256
        s["t_k"], s["t_v"] = B.Transform(C, *_transform(rng, C)), B.Transform(C, *_transform(rng, C))
        # queries share the key blocks of their group of heads, outputs the value blocks
        rep = -(-Q // C)
        for name, key in (("t_q", "t_k"), ("t_o", "t_v")):
            G, P, _ = _transform(rng, C, clip=False)
            s[name] = B.Transform(Q, G, np.concatenate([P] * rep)[: Q // 32], None)
        size = B.batq_code8_bytes if s["bits"] == 8 else B.batq_code_bytes
        for name, t in (("k", s["t_k"]), ("v", s["t_v"])):
            s[name] = _activations(gen, "outliers", M, C).to(torch.bfloat16)
            s[name + "c"], s[name + "s"] = _bytes(size(s["cap"], C)).zero_(), _bytes(B.batq_scale_bytes(s["cap"], C)).zero_()
            B.batq_kv_append(t, _activations(gen, "outliers", L, C).to(torch.bfloat16), s[name + "c"], s[name + "s"], 0,
                             s["cap"], bits=s["bits"])
            s[name + "x"] = torch.empty((L + M, C), dtype=torch.bfloat16, device="cuda")
        s["q"] = torch.randn((M, Q), device="cuda", generator=gen).to(torch.bfloat16)
        s["o"] = torch.randn((M, Q), device="cuda", generator=gen).to(torch.bfloat16)
        s["qt"], s["ot"] = torch.empty_like(s["q"]), torch.empty_like(s["o"])
    else:
        K, N = case["K"], case["N"]
        s["t"] = B.Transform(K, *_transform(rng, K))
        s["kxn"] = case["kxn"]
        s["W"] = (torch.randn((K, N) if case["kxn"] else (N, K), device="cuda", generator=gen) * 0.02).to(_DTYPE[case["w"]])
    return s


def run(s):
    op = s["op"]
    if op == "linear":
        fn = B.batq_linear_a8w4 if s["bits"] == 8 else B.batq_linear
        return fn(s["t"], s["w"], s["X"], Y=s["Y"], workspace=s["ws"])
    if op == "mlp":
        r = B.batq_row_rms_scale(s["X"])
        B.batq_linear_glu(s["t_in"], s["w_in"], s["X"], act_bits=s["bits"], row_scale=r, H=s["H"], workspace=s["ws"])
        B.batq_linear_ex(s["t_down"], s["w_down"], s["H"], act_bits=s["bits"], Y=s["Y"], workspace=s["ws"])
        return s["H"], s["Y"]
    if op == "kv":
        L, n, C = s["L"], s["kx"].shape[0], s["kx"].shape[1]
        for name, t in (("k", s["t_k"]), ("v", s["t_v"])):
            B.batq_kv_append(t, s[name], s[name + "c"], s[name + "s"], L, s["cap"], bits=s["bits"])
            B.batq_kv_dequantize(s[name + "c"], s[name + "s"], s["cap"], 0, n, C, bits=s["bits"], out=s[name + "x"])
        B.batq_transform_apply(s["t_q"], s["q"], B.APPLY_INVERSE_T, out=s["qt"])
        B.batq_transform_apply(s["t_o"], s["o"], B.APPLY_INVERSE, out=s["ot"])
        return {k: s[k] for k in ("kx", "vx", "qt", "ot")}
    w = B.batq_prepare_weight(s["t"], s["W"], w_is_KxN=s["kxn"])
    return w.export()


_MX = {4: 0.5 + 1 / 32, 8: 1.0 + 1 / 32}      # bytes of a quantised element and its share of the scale


def work(case):
    size = {"bf16": 2, "f32": 4}
    if case["op"] == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": M * K * size[case["x"]] + K * N * _MX[4] + M * N * size[case["y"]], "flops": 2.0 * M * K * N}
    if case["op"] == "mlp":
        M, D, F = case["M"], case["D"], case["F"]
        return {"bytes": 2 * M * D * 2 + 3 * D * F * _MX[4] + 2 * M * F, "flops": 6.0 * M * D * F}
    if case["op"] == "kv":
        M, L, C, Q, mx = case["M"], case["context"], case["C"], case["Q"], _MX[case["bits"]]
        # a block's Kronecker product takes 12 multiply-adds per element
        return {"bytes": 2 * (M * C * (2 + mx) + (L + M) * C * (2 + mx) + M * Q * 4), "flops": 24.0 * 2 * M * (C + Q)}
    K, N = case["K"], case["N"]
    return {"bytes": K * N * (size[case["w"]] + _MX[4]), "flops": 24.0 * K * N}


def tolerance(case):
    # Measured against the same path with the transform's sums in fp64 and against fp64 GEMM sums of the same codes:
    # 4-bit layers 0 to 5e-5, 8-bit layers 2e-4 (the matrix instruction's summation window), the MLP block 1e-4 (bf16
    # rounding of the gated activation), the cache 8e-6; the differences are bf16 output roundings and codes at rounding
    # ties.  A single tie in a call of a few rows weighs more than that, hence the common bound.
    if case["op"] == "convert":
        return "exact"                       # bytes, from fp64 products with one rounding
    if case["op"] == "kv":
        return {"rel": 1e-3, "max": 0.5}     # an element at a tie moves by one 4-bit code step
    return {"rel": 1e-3}

"""The calls whose speed users of this library see, with inputs for each: linear layers in ternary-SVD form from one
token to a long prefill, convolutions in ternary-SVD form, and the transition of a dense matrix into that form.

Every case goes through the entry points of paper_2308_07641_amd as a program would: the layer is packed once and kept,
so are the workspace and, where the entry point takes one, the output buffer.  `listed()` holds fixed cases, `draw()`
others from the same ranges.
"""
from __future__ import annotations

import math

import torch

import paper_2308_07641_amd as tsvd

DEV = "cuda:0"
THETA = 0.576           # the threshold angle of the paper's experiments


def _linear(name, M, N, K, B, p0, x_dtype="bf16", y_dtype="f32", x_token_major=False, y_token_major=False, bias=False):
    case = {"op": "linear", "M": M, "N": N, "K": K, "B": B, "p0": p0, "x_dtype": x_dtype, "y_dtype": y_dtype,
            "x_token_major": x_token_major, "y_token_major": y_token_major, "bias": bias}
    return dict(case, name=name) if name else case


def _conv(name, form, c_in, c_out, k, rank, images, H, stride=1, y_dtype="f32", bias=False, groups=1):
    case = {"op": "conv", "form": form, "c_in": c_in, "c_out": c_out, "k": k, "rank": rank, "images": images, "H": H,
            "stride": stride, "y_dtype": y_dtype, "bias": bias, "groups": groups}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest layer, one fp32 vector: what a call costs when there is next to nothing to do
        _linear("tiny", 256, 256, 512, 1, 0.5, x_dtype="f32"),
        # one decoding step of a single sequence through a feed-forward layer of a large language model
        _linear("opt6b7_fc1_decode", 16384, 4096, 8192, 1, 0.6),
        # the same step for a batch of 16 sequences, as a row-per-token program with a bf16 residual stream calls it
        _linear("opt6b7_fc1_decode_b16", 16384, 4096, 8192, 16, 0.6, y_dtype="bf16", x_token_major=True, y_token_major=True, bias=True),
        # a prefill chunk of the same layer
        _linear("opt6b7_fc1_prefill_b256", 16384, 4096, 8192, 256, 0.6, y_dtype="bf16", x_token_major=True, y_token_major=True, bias=True),
        # the prefill of a very large layer: bound by the matrix cores
        _linear("opt66b_fc1_prefill", 36864, 9216, 18432, 2048, 0.6),
        # an encoder's feed-forward layer on one sequence of 512 tokens
        _linear("bert_ffn_in", 3072, 768, 1536, 512, 0.5),
        # a converted layer at a rank that no tile divides, on 16 images of 197 patches, in the layer form
        _linear("ffn_768x3072_rank1545", 3072, 768, 1545, 3152, 0.72, y_dtype="bf16", x_token_major=True, y_token_major=True, bias=True),
        # many positions through a small factorisation (the pointwise layers of a convolutional network, feature-major)
        _linear("convnext_mlp", 2048, 512, 1024, 12544, 0.6),
        # activations that have to stay in fp32, an odd number of them
        _linear("fp32_tokens", 3072, 768, 1536, 197, 0.5, x_dtype="f32", x_token_major=True, y_token_major=True, bias=True),
        # a 3 x 3 convolution whose V takes the taps
        _conv("conv3x3_form0", 0, 256, 256, 3, 768, 32, 14),
        # the depth-wise 7 x 7 layer of a converted network, rank 5 for every channel
        _conv("depthwise7x7", 0, 96, 96, 7, 5, 32, 56, groups=96, y_dtype="bf16", bias=True),
        # converting a matrix: the first 32 components of the transition of a Laplace matrix
        {"name": "transition_laplace_512x256", "op": "transition", "M": 512, "N": 256, "rank": 32, "q": 1},
    ]


def _log(rng, lo, hi):
    """A size spread over the logarithm of lo .. hi; every third one is a multiple of 64 where the range allows."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if v >= 128 and rng.random() < 1 / 3:
        v = max(64, v // 64 * 64)
    return min(max(v, lo), hi)


def draw(rng):
    kind = rng.random()
    if kind < 0.15:
        # convolutions of 64 to 512 channels on planes of 7 to 56
        while True:
            k = rng.choice((3, 3, 5))
            c = _conv(None, rng.randrange(4), _log(rng, 64, 512), _log(rng, 64, 512), k, _log(rng, 64, 1024), _log(rng, 1, 64),
                      rng.choice((7, 14, 28, 56)), rng.choice((1, 1, 2)), rng.choice(("f32", "bf16")), rng.random() < 0.5)
            if c["images"] * c["H"] ** 2 * max(c["c_in"], c["c_out"]) * k * k <= 1 << 27:
                return c
    if kind < 0.25:
        while True:
            c = _log(rng, 64, 768)
            case = _conv(None, 0, c, c, rng.choice((3, 5, 7, 7)), rng.choice((3, 5, 5, 8)), _log(rng, 1, 64), rng.choice((7, 14, 28, 56)),
                         rng.choice((1, 1, 1, 2)), rng.choice(("f32", "bf16")), rng.random() < 0.5, groups=c)
            if case["images"] * case["H"] ** 2 * c <= 1 << 25:
                return case
    if kind < 0.35:
        while True:
            M, N, q, rank = _log(rng, 96, 768), _log(rng, 96, 768), rng.choice((1, 1, 2, 4)), rng.randint(6, 40)
            if M * N * rank <= 512 * 256 * 32:
                return {"op": "transition", "M": M, "N": N, "rank": rank, "q": q}
    while True:
        M, N = _log(rng, 192, 16384), _log(rng, 96, 8192)
        K = _log(rng, 64, min(8192, 2 * max(M, N)))
        x_dtype = "f32" if rng.random() < 0.2 else "bf16"
        band = rng.random()
        B = 1 if band < 0.2 else _log(rng, 2, 16) if band < 0.4 else _log(rng, 17, 512) if band < 0.7 else _log(rng, 513, 16384)
        if K * (M + N) > 8192 * (16384 + 4096) or max(M, N, K) * B > 1 << 26 or K * (M + N) * B > 1 << 39:
            continue
        form = rng.random() < 0.5       # the layer form: rows are tokens
        return _linear(None, M, N, K, B, rng.choice((0.5, 0.6, 0.72)), x_dtype, rng.choice(("f32", "bf16")) if form else "f32", form, form,
                       form and rng.random() < 0.7)


# ---- inputs ------------------------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _ternary(rows, cols, p0, g):
    """Entries 0 with probability p0 (to 1/128), +1 and -1 alike; int8 on the host, as tsvd_pack takes them."""
    r = torch.randint(0, 256, (rows, cols), generator=g, device=DEV, dtype=torch.uint8)
    half = int(round((1.0 - p0) * 128))
    return ((r < half).to(torch.int8) - (r >= 256 - half).to(torch.int8)).cpu().numpy()


def _scales(K, g):
    return (torch.randn(K, generator=g, device=DEV).abs() * 0.02).cpu().numpy()


def _torch_dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _prepare_linear(c, g):
    M, N, K, B = c["M"], c["N"], c["K"], c["B"]
    h = tsvd.tsvd_pack(_ternary(M, K, c["p0"], g), _scales(K, g), _ternary(K, N, c["p0"], g))
    # normally distributed activations, some features an order of magnitude above the rest as in transformers
    x = torch.randn((B, N), generator=g, device=DEV)
    x *= torch.where(torch.rand(N, generator=g, device=DEV) < 0.01, 20.0, 1.0)
    x = x.to(_torch_dtype(c["x_dtype"]))
    if not c["x_token_major"]:
        x = x.t().contiguous() if B > 1 else x.reshape(N)       # (a single token is a vector)
    code = tsvd.TSVD_BF16 if c["x_dtype"] == "bf16" else tsvd.TSVD_F32
    xl = tsvd.TSVD_TOKEN_MAJOR if c["x_token_major"] else tsvd.TSVD_FEATURE_MAJOR
    return {"op": "layer" if c["x_token_major"] else "linear", "h": h, "x": x,
            "y": torch.empty((B, M) if c["y_token_major"] else (M, B), dtype=_torch_dtype(c["y_dtype"]), device=DEV),
            "bias": torch.randn(M, generator=g, device=DEV) if c["bias"] else None,
            "y_dtype": tsvd.TSVD_BF16 if c["y_dtype"] == "bf16" else tsvd.TSVD_F32,
            "workspace": torch.empty(tsvd.tsvd_workspace_bytes_ex(h, B, code, xl), dtype=torch.uint8, device=DEV)}


def _conv_matrices(c):
    """(rows of U, columns of V) of the packed matrix."""
    k, f = c["k"], c["form"]
    u, v = {0: (1, k * k), 1: (k * k, 1), 2: (k, k), 3: (k, k)}[f]
    return c["c_out"] * u, c["c_in"] // c["groups"] * v


def _prepare_conv(c, g):
    rows, cols = _conv_matrices(c)
    G, rank = c["groups"], c["rank"]
    if G > 1:                       # rank factors for each channel, side by side; a row of U uses its own channel's only
        own = torch.arange(c["c_out"], device=DEV).repeat_interleave(rank)
        U = torch.zeros((rows, rank * G), dtype=torch.int8, device=DEV)
        sign = torch.randint(0, 2, (rank * G,), generator=g, device=DEV, dtype=torch.int8) * 2 - 1
        U[own, torch.arange(rank * G, device=DEV)] = sign
        U, p0 = U.cpu().numpy(), 0.765
    else:
        U, p0 = _ternary(rows, rank, 0.7, g), 0.7
    h = tsvd.tsvd_pack(U, _scales(rank * G, g), _ternary(rank * G, cols, p0, g))
    x = torch.randn((c["c_in"], c["images"], c["H"], c["H"]), generator=g, device=DEV).to(torch.bfloat16)
    return {"op": "conv", "h": h, "x": x, "form": c["form"], "c_in": c["c_in"], "c_out": c["c_out"], "k": c["k"], "stride": c["stride"],
            "groups": G, "bias": torch.randn(c["c_out"], generator=g, device=DEV) if c["bias"] else None,
            "y_dtype": tsvd.TSVD_BF16 if c["y_dtype"] == "bf16" else tsvd.TSVD_F32}


def prepare(case, seed):
    g = _generator(seed)
    if case["op"] == "linear":
        return _prepare_linear(case, g)
    if case["op"] == "conv":
        return _prepare_conv(case, g)
    u = torch.rand((case["M"], case["N"]), generator=g, device=DEV, dtype=torch.float64) - 0.5
    W = -torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.4999999999))       # Laplace
    return {"op": "transition", "W": W, "rank": case["rank"], "q": case["q"]}


def run(s):
    if s["op"] == "linear":
        return tsvd.tsvd_forward(s["h"], s["x"], s["y"], workspace=s["workspace"])
    if s["op"] == "layer":
        return tsvd.tsvd_forward_io(s["h"], s["x"], tsvd.TSVD_TOKEN_MAJOR, s["bias"], s["y"], s["y_dtype"], tsvd.TSVD_TOKEN_MAJOR,
                                    workspace=s["workspace"])
    if s["op"] == "conv":
        k, st, pad = s["k"], s["stride"], s["k"] // 2
        return tsvd.tsvd_conv2d_forward(s["h"], s["form"], s["c_in"], s["c_out"], k, k, s["x"], (st, st), (pad, pad), bias=s["bias"],
                                        y_dtype=s["y_dtype"], groups=s["groups"])
    U, S, V, errors, status = tsvd.tsvd_transition(s["W"], THETA, 0.0, s["rank"], q=s["q"])
    return {"U": U, "S": S, "V": V, "errors": torch.tensor(errors, dtype=torch.float64), "status": status}


# ---- what a pass cannot do without ---------------------------------------------------------------------------------
def _size(dtype):
    return 2 if dtype == "bf16" else 4


def work(case):
    """Packed codes (2 bits each), scales, activations and results once; a multiplication and an addition for every code and column.
    A depth-wise layer: those of its own taps.  A component of the transition: two products with the residual for its singular
    pair, the right side of its scale, and the update of the residual, in fp64."""
    if case["op"] == "linear":
        M, N, K, B = case["M"], case["N"], case["K"], case["B"]
        return {"bytes": K * (M + N) / 4 + 4 * K + N * B * _size(case["x_dtype"]) + M * B * _size(case["y_dtype"]) + (4 * M if case["bias"] else 0),
                "flops": 2 * K * (M + N) * B}
    if case["op"] == "conv":
        c, k = case, case["k"]
        out = (c["H"] + 2 * (k // 2) - k) // c["stride"] + 1
        rows, cols = _conv_matrices(c)
        # positions at which V and U are applied: form 1 keeps the input plane between them, forms 2 and 3 reduce one dimension
        between = {0: out * out, 1: c["H"] ** 2, 2: c["H"] * out, 3: out * c["H"]}[c["form"]]
        K = c["rank"] * c["groups"]
        codes = K * cols + (c["c_out"] * c["rank"] if c["groups"] > 1 else rows * K)
        flops = 2 * c["images"] * (between * K * cols + (out * out * c["c_out"] * c["rank"] if c["groups"] > 1 else out * out * K * rows))
        data = 2 * c["c_in"] * c["images"] * c["H"] ** 2 + _size(c["y_dtype"]) * c["c_out"] * c["images"] * out * out
        return {"bytes": codes / 4 + 4 * K + data, "flops": flops}
    M, N, r = case["M"], case["N"], case["rank"]
    return {"bytes": 8 * M * N + (M + N) * r + 16 * r, "flops": 8 * M * N * r}


def tolerance(case):
    if case["op"] == "transition":
        # fp64 throughout; the vectors are converged to 1e-12 of sigma over the gap to the next singular value
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    if case["y_dtype"] == "bf16":
        return {"rel": 4e-3, "max": 1e-2}           # one rounding to 8 bits
    if case["op"] == "linear" and (case["B"] == 1 or case["x_dtype"] == "f32") or case["op"] == "conv" and case["groups"] > 1:
        return {"rel": 1e-5, "max": 1e-4}           # fp32 sums
    return {"rel": 5e-4, "max": 4e-3}               # bf16 activations, the intermediate vector held to 11 bits

"""The workloads that this library is timed on: what its users call, over the range of sizes they call it with.

A case is one call (a training step: one forward and one backward call) of the public entry points on device
tensors that are already in place.  The listed cases are the repository's five benchmark configurations and the
calls around them: short and ragged sequences, prompts, one decoded token, fp32, the bidirectional training step,
and the feature map by itself.  `draw` gives further sizes of the same kinds.
"""
import math

import torch

import paper_2603_04127_amd as dk

# Value distributions of the benchmark configurations: the spectrum of the query/key covariance and the
# condition number of M (None: M = I + 0.1 N(0, 1)).
_LOG = ("log", 100.0, 0.01, 10.0)     # encoder, long context, fine-tuning
_MILD = ("log", 10.0, 0.1, None)      # fp32
_TOP = ("top", 8, 0.9, 20.0)          # causal prefill, decode


def _case(name, kind, B, H, L, d, m, dtype, **more):
    c = {"kind": kind, "B": B, "H": H, "L": L, "d": d, "m": m, "dtype": dtype, "shared_w": False, "out_f32": False}
    c.update(more)
    return {"name": name, **c} if name else c


def listed():
    return [
        # The smallest problem: one head, one short sequence; launches and latency are all there is.
        _case("tiny_f32", "bidir", 1, 1, 256, 64, 64, "f32"),
        # An fp32 encoder layer (evaluation at full precision).
        _case("encoder_f32", "bidir", 2, 12, 1024, 64, 256, "f32"),
        # A small fp32 causal training step on a ragged sequence.
        _case("finetune_f32", "train_causal", 1, 8, 1000, 64, 128, "f32"),
        # The encoder layer of the headline benchmark.
        _case("encoder_bf16", "bidir", 8, 12, 4096, 64, 256, "bf16"),
        # The same layer on a small batch of short sentences of no round length.
        _case("encoder_short_bf16", "bidir", 3, 12, 509, 64, 256, "bf16"),
        # Long context, many features: the largest single call.
        _case("long_bf16", "bidir", 1, 8, 131072, 64, 512, "bf16"),
        # Decoder prefill of a batch.
        _case("prefill_bf16", "causal", 4, 16, 8192, 128, 256, "bf16"),
        # Prefill of one user's prompt.
        _case("prompt_bf16", "causal", 1, 16, 777, 128, 256, "bf16"),
        # One decoded token for a serving batch.
        _case("decode_bf16", "decode", 8, 16, 1, 128, 256, "bf16"),
        # Fine-tuning step of a decoder layer: forward and backward.
        _case("finetune_causal_bf16", "train_causal", 2, 12, 4096, 64, 256, "bf16"),
        # Fine-tuning step of an encoder layer: forward and backward.
        _case("finetune_bidir_bf16", "train_bidir", 2, 12, 2048, 64, 256, "bf16"),
        # The feature map alone, queries and keys (estimator studies, callers with a linear attention of their own).
        _case("featurize_bf16", "featurize", 8, 12, 1024, 64, 256, "bf16"),
    ]


# kind, dtype -> (d, m) pairs, shortest sequence, most positions over all heads (each the listed kind's largest)
_RANGES = [
    ("bidir", "f32", ((64, 64), (64, 128), (64, 256)), 33, 24 * 1024),
    ("train_causal", "f32", ((64, 64), (64, 128)), 33, 8000),
    ("bidir", "bf16", ((64, 256), (64, 512), (128, 256)), 33, 393216),
    ("causal", "bf16", ((64, 256), (128, 256)), 17, 524288),
    ("decode", "bf16", ((64, 256), (128, 256)), 1, 128),
    ("train_causal", "bf16", ((64, 256),), 65, 98304),
    ("train_bidir", "bf16", ((64, 256),), 65, 49152),
    ("featurize", "bf16", ((64, 256), (64, 512)), 33, 98304),
]


def draw(rng):
    kind, dtype, shapes, shortest, most = rng.choice(_RANGES)
    d, m = rng.choice(shapes)
    if kind == "featurize" and m > 256:
        most //= 2
    while True:
        B, H = rng.choice((1, 1, 2, 3, 4, 6, 8)), rng.choice((1, 2, 4, 6, 8, 12, 16))
        if B * H * shortest <= most:
            break
    longest = most // (B * H)
    L = 1 if kind == "decode" else int(round(math.exp(rng.uniform(math.log(shortest), math.log(longest)))))
    attention = kind in ("bidir", "causal")
    return _case(None, kind, B, H, L, d, m, dtype, shared_w=rng.random() < 0.2,
                 out_f32=attention and dtype == "bf16" and rng.random() < 0.2)


def _haar(n, count, gen):
    q, r = torch.linalg.qr(torch.randn(count, n, n, generator=gen, dtype=torch.float64))
    return q * torch.sign(torch.diagonal(r, dim1=-2, dim2=-1))[:, None, :]


def _spectrum(d, dist):
    if dist[0] == "log":
        return torch.logspace(math.log10(dist[1]), math.log10(dist[2]), d, dtype=torch.float64)
    k, share = dist[1], dist[2]
    s = torch.full((d,), (1.0 - share) * d / (d - k), dtype=torch.float64)
    s[:k] = share * d / k
    return s


def _distribution(case):
    if case["dtype"] == "f32":
        return _MILD
    return _TOP if case["kind"] in ("causal", "decode") else _LOG


def prepare(case, seed):
    B, H, L, d, m = (case[k] for k in ("B", "H", "L", "d", "m"))
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    dist = _distribution(case)
    host = torch.Generator().manual_seed(1000003 * seed + 17)
    dev = torch.Generator(device="cuda").manual_seed(1000003 * seed + 29)
    colour = (_spectrum(d, dist).sqrt()[None, :, None] * _haar(d, H, host).transpose(1, 2)).float().cuda()
    if dist[3] is None:
        M = torch.eye(d) + 0.1 * torch.randn(H, d, d, generator=host)
    else:
        sigma = torch.logspace(0.0, -math.log10(dist[3]), d, dtype=torch.float64)
        M = ((_haar(d, H, host) * sigma[None, None, :]) @ _haar(d, H, host).transpose(1, 2)).float()
    W = torch.randn(*((m, d) if case["shared_w"] else (H, m, d)), generator=host)

    def rows(n):
        return torch.matmul(torch.randn(B, H, n, d, generator=dev, device="cuda"), colour)

    def white(n):
        return torch.randn(B, H, n, d, generator=dev, device="cuda")

    s = {"case": case, "M": M.cuda().contiguous(), "W": W.cuda().contiguous()}
    if case["kind"] == "decode":
        s.update(q=rows(1)[:, :, 0].to(dtype).contiguous(), k=rows(1)[:, :, 0].to(dtype).contiguous(),
                 v=white(1)[:, :, 0].to(dtype).contiguous(), state=_past(s, rows(64), white(64)))
        return s
    s["Q"], s["K"] = rows(L).to(dtype).contiguous(), rows(L).to(dtype).contiguous()
    if case["kind"] != "featurize":
        s["V"] = white(L).to(dtype).contiguous()
    if case["kind"].startswith("train"):
        s["dOut"] = white(L).to(dtype).contiguous()
    return s


def _past(s, K, V):
    """The recurrent state after the tokens (K, V), as dark_decode_step keeps it."""
    W = s["W"] if s["W"].dim() == 3 else s["W"].expand(s["M"].shape[0], *s["W"].shape)
    x = torch.matmul(K * K.shape[-1] ** -0.25, s["M"].transpose(1, 2).contiguous())
    logit = torch.matmul(x, W.transpose(1, 2).contiguous()) - 0.5 * x.square().sum(-1, keepdim=True)
    c = logit.amax(dim=(2, 3))
    phi = torch.exp(logit - c[:, :, None, None])
    S = torch.matmul(phi.transpose(2, 3).contiguous(), V).contiguous()
    return S, phi.sum(2).contiguous(), c.contiguous()


def run(state):
    case, M, W = state["case"], state["M"], state["W"]
    kind = case["kind"]
    if kind == "decode":
        out = dk.dark_decode_step(state["q"], state["k"], state["v"], M, W, state["state"])
        return out, state["state"]
    Q, K = state["Q"], state["K"]
    if kind == "featurize":
        return dk.dark_featurize(Q, M, W, True), dk.dark_featurize(K, M, W, False)
    V = state["V"]
    out_dtype = torch.float32 if case["out_f32"] else None
    if kind == "bidir":
        return dk.dark_attn_fwd(Q, K, V, M, W, out_dtype=out_dtype)
    if kind == "causal":
        return dk.dark_attn_causal_fwd(Q, K, V, M, W, out_dtype=out_dtype)
    if kind == "train_causal":
        out, saved = dk.dark_attn_causal_fwd_save(Q, K, V, M, W)
        return out, dk.dark_attn_bwd(Q, K, V, M, W, state["dOut"], True, saved=saved)
    out = dk.dark_attn_fwd(Q, K, V, M, W)
    return out, dk.dark_attn_bwd(Q, K, V, M, W, state["dOut"], False)


def work(case):
    B, H, L, d, m = (case[k] for k in ("B", "H", "L", "d", "m"))
    n, size = B * H * L, 4 if case["dtype"] == "f32" else 2
    weights = 4 * (H * d * d + (1 if case["shared_w"] else H) * m * d)
    project = 2 * d * m + 2 * d * d      # one row: its logits and its norm term
    if case["kind"] == "decode":
        return {"bytes": weights + n * (4 * d * size + 2 * 4 * (m * (d + 1) + 1)), "flops": n * (2 * project + 4 * m * (d + 1))}
    if case["kind"] == "featurize":
        return {"bytes": weights + 2 * n * (d + m) * size + 4 * (n + B * H), "flops": 2 * n * project}
    forward = n * (4 * d * m + 2 * d * d + 4 * m * (d + 1))   # the norm terms of the queries cancel
    if not case["kind"].startswith("train"):
        return {"bytes": weights + n * d * (3 * size + (4 if case["out_f32"] else size)), "flops": forward}
    # every contraction of the forward pass has two gradient contractions of its size
    return {"bytes": weights + n * d * (5 * size + 3 * 4) + 4 * H * d * d, "flops": 3 * forward}


def tolerance(case):
    # About four times the largest error against the same computation in fp64 over the listed cases and some thirty
    # drawn ones.  The bf16 figures are those of bf16 operands (2^-9 each) and, in the training step, of gradients
    # that are differences of large terms; "max" is a small coordinate beside a row of ordinary size.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 3e-4}            # measured 2.4e-6, 7e-5
    if case["kind"] in ("decode", "featurize"):
        return {"rel": 8e-3, "max": 5e-2}            # measured 1.9e-3, 1.1e-2
    if case["kind"] == "train_causal":
        return {"rel": 2e-2, "max": 0.9}             # measured 5.5e-3, 0.25
    return {"rel": 1.5e-2, "max": 0.25}              # measured 3.8e-3, 6.5e-2

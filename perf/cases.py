"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values:
  kind       "core"  the attention core on (B, H, n, d) tensors
             "block" the attention block on (B, n, H * d) tensors, with its four projections
             "haar"  the gated Haar filter alone (the stage entry point)
  backward   False: the forward pass (inference); True: forward and backward (one training step)
  dtype      "bf16" or "f32" (storage of the large tensors)
  B H n d L m, and for the core
  layout     "bhnd": dense (B, H, n, d); "bnhd": heads side by side as a projection leaves them
  alg1       True: the options of the paper's Algorithm 1 (LayerNorm output stage, gate pooled over
             the heads, separate random matrices for queries and keys)

Sizes are those of the five benchmark configurations, of the paper's own models (two levels, 1024
random features, head dimensions 16 and 32) and of the tests.
"""
import math

import torch

from paper_2507_08637_amd import autograd, binding

# B * H * n * d * m of the largest core case: the long sequence, the paper's text classifier and its
# 128k-token classifier all have this much, and no drawn case has more.
MOST_CORE = 8 * 131072 * 64 * 256
# elements of the largest tensor that the filter stage is given
MOST_HAAR = 8 * 131072 * 64


def _core(name, dtype, backward, B, H, n, d, L, m, layout="bhnd", alg1=False):
    return dict(name=name, kind="core", dtype=dtype, backward=backward, B=B, H=H, n=n, d=d, L=L, m=m,
                layout=layout, alg1=alg1)


def _block(name, backward, B, H, n, d, L, m):
    return dict(name=name, kind="block", dtype="bf16", backward=backward, B=B, H=H, n=n, d=d, L=L, m=m)


def listed():
    return [
        # the smallest call: one short float32 sequence, one head; latency and launches count
        _core("infer_f32_n1024", "f32", False, 1, 1, 1024, 64, 3, 64),
        # a training step on two short sequences of no round length, heads side by side as the
        # projections of a model leave them
        _core("train_bf16_n1000", "bf16", True, 2, 4, 1000, 64, 4, 256, layout="bnhd"),
        # inference on a batch of ordinary sequences
        _core("infer_bf16_n4096", "bf16", False, 8, 8, 4096, 64, 4, 128),
        # a training step of an ordinary model on 16k tokens
        _core("train_bf16_n16384", "bf16", True, 4, 12, 16384, 64, 5, 256),
        # the headline: a training step on one sequence of 131072 tokens
        _core("train_bf16_n131072", "bf16", True, 1, 8, 131072, 64, 6, 256),
        # a transform whose depth grows with the sequence (L of order log n), last block partial
        _core("train_bf16_deep_n30000", "bf16", True, 1, 8, 30000, 64, 10, 256),
        # the paper's Algorithm 1 as it is written, head dimension 128
        _core("train_bf16_alg1_n4096", "bf16", True, 2, 8, 4096, 128, 6, 512, alg1=True),
        # the paper's text classifier: 32 reviews of 4000 tokens, four heads of 32, in float32
        _core("train_f32_n4000_d32", "f32", True, 32, 4, 4000, 32, 2, 1024),
        # the paper's 128k-token classifier: two sequences, four heads of 16
        _core("train_bf16_n131072_d16", "bf16", True, 2, 4, 131072, 16, 2, 1024),
        # the attention block of a small model at inference
        _block("block_infer_n2048", False, 1, 8, 2048, 64, 5, 256),
        # the attention block of a large model: a training step, hidden 2048, 131072 tokens
        _block("block_train_n65536", True, 2, 16, 65536, 128, 6, 512),
        # the filter stage on its own, on the queries of the headline case
        dict(name="haar_bf16_n131072", kind="haar", dtype="bf16", backward=False, B=1, H=8, n=131072, d=64, L=6, m=16,
             layout="bhnd"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["core", "block", "haar"], [16, 3, 2])[0]
    if kind == "haar":
        d = rng.choice([16, 32, 48, 64, 96, 128])
        n = _log_int(rng, 1000, 131072)
        slices = min(_log_int(rng, 4, 256), MOST_HAAR // (n * d))
        H = rng.choice([h for h in (1, 2, 4, 8) if h <= max(1, slices)])
        return dict(kind="haar", dtype=rng.choice(["bf16", "bf16", "f32"]), backward=False, B=max(1, slices // H), H=H, n=n,
                    d=d, L=rng.randint(1, min(10, n.bit_length() - 1)), m=16, layout=rng.choice(["bhnd", "bnhd"]))
    if kind == "block":
        d = rng.choice([64, 64, 128])
        hidden = rng.choice([512, 1024, 1024, 2048])
        n = 256 * _log_int(rng, 4, 256)
        B = rng.randint(1, max(1, min(8, 131072 // n)))
        return dict(kind="block", dtype="bf16", backward=rng.random() < 0.5, B=B, H=hidden // d, n=n, d=d,
                    L=rng.randint(2, 6), m=rng.choice([128, 256, 512]))
    # head dimensions 64 and 128 in bf16 are most of the use; 16 and 32 are the paper's own models
    d = rng.choices([16, 32, 64, 128], [2, 3, 8, 3])[0]
    dtype = rng.choices(["bf16", "f32"], [3, 1])[0]
    m = rng.choice([512, 1024]) if d <= 32 else rng.choice([128, 256, 256, 512])
    n = _log_int(rng, 1000, 131072)
    H = rng.choice([1, 2, 4, 8, 12])
    B = min(_log_int(rng, 1, 64), MOST_CORE // (H * n * d * m))
    while B < 1:
        H = H // 2
        B = MOST_CORE // (max(H, 1) * n * d * m)
        if H <= 1 and B < 1:   # d * m at its largest: one head of as many tokens as are allowed
            n, B = MOST_CORE // (d * m), 1
    return dict(kind="core", dtype=dtype, backward=rng.random() < 0.65, B=B, H=max(H, 1), n=n, d=d,
                L=rng.randint(2, 6) if rng.random() < 0.8 else rng.randint(7, min(12, n.bit_length() - 1)), m=m,
                layout=rng.choice(["bhnd", "bnhd"]), alg1=rng.random() < 0.15)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def prepare(case, seed):
    """Inputs and parameters.  Rows are tokens of a sequence that has a course in time: noise of its
    own per token, on slow waves that all tokens share, so that the wavelet scales (and with them the
    gradients of the gate's parameters) carry something other than noise.  The values follow three
    column profiles with their own waves, and the incoming gradient is noise on similar ones."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(seed)
    B, H, n, d, L, m = (case[k] for k in ("B", "H", "n", "d", "L", "m"))
    dt = _dtype(case)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32)

    t = torch.arange(n, device=dev, dtype=torch.float32)

    def wave(period, shift=0.0):
        return torch.sin(2 * math.pi * t / period + shift)

    state = dict(case=case, L=L)
    if case["kind"] == "haar":
        x = _lay(case, 0.5 * normal(B, H, n, d) + 1.5 * wave(256)[:, None], dt)
        state.update(x=x, filt=1.0 + 0.3 * normal(B * H, L + 1))
        return state

    state.update(
        sigma=1.0 + 0.1 * normal(1).clamp(-3, 3),
        gate_w=normal(H, L + 1, d) / math.sqrt(d),
        gate_b=0.5 * normal(H, L + 1),
        scale_w=1.0 + 0.1 * normal(L + 1),
        omega=normal(*((2, d, m) if case.get("alg1") else (d, m))).to(dt))
    xj = 2 * math.pi * torch.arange(d, device=dev, dtype=torch.float32) / d
    vals = (wave(256)[:, None] * torch.cos(xj) + wave(128, math.pi / 2)[:, None] * torch.sin(xj)
            + 0.7 * wave(512)[:, None] * torch.cos(2 * xj) + torch.cos(3 * xj))
    back = (wave(256, 0.6)[:, None] * torch.cos(xj + 0.4) + 0.7 * wave(128, 1.2)[:, None] * torch.sin(xj + 0.4)
            + 0.5 * torch.cos(2 * xj))
    if case["kind"] == "core":
        q = normal(B, H, n, d) + (0.7 * wave(256) + 0.2)[:, None]
        k = normal(B, H, n, d) + (0.7 * wave(256) + 0.2)[:, None]
        v = 0.3 * normal(B, H, n, d) + vals
        state.update(q=_lay(case, q, dt), k=_lay(case, k, dt), v=_lay(case, v, dt))
        if case["backward"]:
            state["dout"] = _lay(case, 0.3 * normal(B, H, n, d) + back, dt)
            for name in ("q", "k", "v", "sigma", "gate_w", "gate_b", "scale_w"):
                state[name].requires_grad_(True)
        return state

    # block: token features are noise plus a wave along a direction of the model; the projections'
    # weights have the usual 1 / sqrt(hidden) scale, and the wave comes out of each of them
    hidden = H * d
    unit = torch.ones(hidden, device=dev)
    x = torch.empty(B, n, hidden, device=dev, dtype=dt)
    for b in range(B):
        x[b] = normal(n, hidden) + (1.5 * wave(256) + 0.3)[:, None] * unit
    state["x"] = x
    one = torch.ones(hidden, hidden, device=dev) / hidden
    for name, columns in (("wq", unit), ("wk", unit), ("wv", torch.cos(xj).repeat(H)), ("wo", None)):
        w = normal(hidden, hidden) / (2 * math.sqrt(hidden))
        state[name] = (w if columns is None else w + one * columns).to(dt)
    if case["backward"]:
        dy = torch.empty(B, n, hidden, device=dev, dtype=dt)
        for b in range(B):
            dy[b] = 0.3 * normal(n, hidden) + back.repeat(1, H)
        state["dy"] = dy
        for name in ("x", "wq", "wk", "wv", "wo", "sigma", "gate_w", "gate_b", "scale_w"):
            state[name].requires_grad_(True)
    return state


def _lay(case, x, dt):
    """(B, H, n, d) in the case's memory layout and dtype."""
    if case["layout"] == "bnhd":
        return x.permute(0, 2, 1, 3).to(dt).contiguous().permute(0, 2, 1, 3)
    return x.to(dt)


ALG1 = binding.FLAG_LAYERNORM | binding.FLAG_POOLED_GATE | binding.FLAG_SEPARATE_OMEGA
ALG1_EPS = 1e-3   # of the LayerNorm


def run(state):
    case, L = state["case"], state["L"]
    if case["kind"] == "haar":
        return binding.wersa_haar_filter(state["x"], state["filt"], L)
    params = tuple(state[k] for k in ("omega", "sigma", "gate_w", "gate_b", "scale_w"))
    if case["kind"] == "block":
        weights = tuple(state[k] for k in ("wq", "wk", "wv", "wo"))
        if not case["backward"]:
            y, _ = binding.wersa_block_forward(state["x"], *weights, case["H"], *params, L)
            return y
        y = autograd.wersa_attention_block(state["x"], *weights, case["H"], *params, L)
        return (y.detach(),) + torch.autograd.grad(y, (state["x"],) + weights + params[1:], state["dy"])
    qkv = (state["q"], state["k"], state["v"])
    if case["alg1"]:   # the options go through the calls that take flags
        opt = dict(eps=ALG1_EPS, flags=ALG1)
        with torch.no_grad():
            out, saved = binding.wersa_forward(*qkv, *params, L, **opt)
            if not case["backward"]:
                return out
            grads = binding.wersa_backward(*qkv, *params, out, state["dout"], saved, L, **opt)
        return dict(grads, out=out)
    if not case["backward"]:
        return binding.wersa_forward(*qkv, *params, L)[0]
    out = autograd.wersa_attention(*qkv, *params, L)
    return (out.detach(),) + torch.autograd.grad(out, qkv + params[1:], state["dout"])


def work(case):
    """Contractions of n x d x m per slice: projection of Q and of K, key-value product, apply (4);
    backward: the two projections again, dPhi, dX_F and the m x d product of each side (8).  Bytes: every
    tensor that comes in once and every tensor that goes out once."""
    B, H, n, d, L, m = (case[k] for k in ("B", "H", "n", "d", "L", "m"))
    e = 4 if case["dtype"] == "f32" else 2
    tensor = B * H * n * d * e
    if case["kind"] == "haar":
        return {"bytes": 2 * tensor, "flops": 2 * B * H * n * d * (L + 1)}
    contraction = 2 * B * H * n * d * m
    params = 4 * (H * (L + 1) * (d + 1) + L + 2) + d * m * e * (2 if case.get("alg1") else 1)
    flops = contraction * (12 if case["backward"] else 4)
    if case["kind"] == "core":   # q, k, v -> out; q, k, v, dout -> out, dq, dk, dv
        return {"bytes": tensor * (8 if case["backward"] else 4) + params * (2 if case["backward"] else 1), "flops": flops}
    hidden = H * d
    product = 2 * B * n * hidden * hidden   # four projections; two products each in the backward
    weights = 4 * hidden * hidden * e
    return {"bytes": tensor * (4 if case["backward"] else 2) + weights * (2 if case["backward"] else 1) + params,
            "flops": flops + product * (12 if case["backward"] else 4)}


def tolerance(case):
    """float32, forward: sums of up to some thousand terms in another order.  float32, backward: a
    pre-activation X_F Omega that lies within a few rounding errors (2^-24 relative) of zero may fall on
    the other side of the ReLU's step, which changes one of about m / 2 terms of a row by its whole
    size: a share of about 2e-7 of the elements, each worth 2 / m of its row's squared norm, is
    sqrt(4e-7) = 6e-4 over the tensor and up to some tenths of the root mean square in one row.
    bf16: outputs rounded to 8 bits; backward: the same effect at the 11 bits that the projection's
    operands have (6e-3 to 9e-3 against exact arithmetic, so up to 1.3e-2 between two implementations),
    and parameter gradients that are sums over such tensors."""
    if case["kind"] == "haar":
        return {"rel": 1e-6, "max": 1e-5} if case["dtype"] == "f32" else {"rel": 3e-3, "max": 2e-2}
    if case["dtype"] == "f32":
        return {"rel": 1e-3, "max": 0.9} if case["backward"] else {"rel": 1e-5, "max": 1e-3}
    return {"rel": 2e-2, "max": 0.99} if case["backward"] else {"rel": 6e-3, "max": 0.2}

"""What a user of the library has it do, as cases that can be timed and compared: decoding, prefill, training and the
whole layer around the delta rule, through the functions of `paper_2605_05838_amd.binding`.

A case names its kind and its sizes.  Shapes: the five measurement configurations (`synth.CONFIGS`: 2, 8 or 16 heads of
64 or 128, up to 32 768 tokens), the decode, hand-off, packed and layer workloads of `bench.py`, and the odd lengths of
the tests.  Values follow `synth`: L2-normalised q and k, sigmoid step sizes, slowly decaying gates.
"""
import math
import random

import torch

from paper_2605_05838_amd import binding

NAMES = ("q", "k", "v", "beta", "alpha", "mu")


def listed():
    return [
        # one sequence being generated, one token per call: the smallest call there is, all latency
        dict(name="decode_one", kind="decode", B=1, T=1, H=16, d=128, dtype="bf16"),
        # a full serving batch, one token per sequence and call: every call reads and writes 512 MB of states twice
        dict(name="decode_batch", kind="decode", B=256, T=1, H=16, d=128, dtype="bf16"),
        # one prompt of ordinary, odd length before its decoding starts (time to first token)
        dict(name="prefill_prompt", kind="prefill", B=1, T=777, H=16, d=128, dtype="bf16"),
        # a batch of equal prompts / an evaluation forward at the 400M layer shape
        dict(name="prefill_batch", kind="prefill", B=8, T=2048, H=8, d=128, dtype="bf16"),
        # prompts of mixed lengths packed into one call, their final states wanted for decoding
        dict(name="packed_prefill", kind="packed_prefill", T=16384, n=24, H=16, d=128, dtype="bf16", carry=False, lens=1),
        # the same for sequences that go on from states they already have (chunked prefill, next turn of a conversation)
        dict(name="packed_continue", kind="packed_prefill", T=8192, n=24, H=16, d=128, dtype="bf16", carry=True, lens=2),
        # the training step of the 1.3B layer shape, forward keeping what the backward can use
        dict(name="train_layer_shape", kind="train", B=4, T=4096, H=16, d=128, dtype="bf16", keep=True, eta=False,
             segment=False),
        # training on one long document
        dict(name="train_long", kind="train", B=1, T=32768, H=16, d=128, dtype="bf16", keep=True, eta=False, segment=False),
        # one segment of a longer sequence of odd length: states in, adjoints of the final states in, memory-lean forward
        dict(name="train_segment", kind="train", B=3, T=1500, H=8, d=64, dtype="bf16", keep=False, eta=True, segment=True),
        # 32-bit storage, small: how a model is checked against a reference before it is trained
        dict(name="train_f32", kind="train", B=2, T=1024, H=4, d=64, dtype="f32", keep=True, eta=True, segment=False),
        # a training batch of documents packed into one row
        dict(name="packed_train", kind="packed_train", T=32768, n=64, H=16, d=128, dtype="bf16", lens=3),
        # the whole layer around the delta rule, forward and backward: gates, front end, chunkwise rule, back end
        dict(name="layer_step", kind="layer", B=4, T=2048, H=16, d=128, dtype="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("decode", "prefill", "packed_prefill", "train", "packed_train", "layer"))
    H, d = rng.choice((4, 8, 16)), rng.choice((64, 128, 128))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f32")) if kind in ("decode", "prefill", "train") else "bf16"
    # (token, head) pairs of a case: the fp32 matrix rate is a sixteenth of the bf16 one
    most = 32768 if dtype == "f32" else 262144
    if kind == "decode":
        return dict(kind=kind, B=_log(rng, 1, 256), T=rng.choice((1, 1, 1, 2, 4, 8)), H=H, d=d, dtype=dtype)
    if kind == "prefill":
        B = rng.randint(1, 8)
        return dict(kind=kind, B=B, T=_log(rng, 16, most // (B * H)), H=H, d=d, dtype=dtype)
    if kind == "packed_prefill":
        T = _log(rng, 256, most // H)
        return dict(kind=kind, T=T, n=_log(rng, 1, max(2, min(48, T // 16))), H=H, d=d, dtype=dtype, carry=rng.random() < 0.5,
                    lens=rng.randint(1, 10 ** 6))
    if kind == "packed_train":
        T = _log(rng, 512, 2 * most // H)
        return dict(kind=kind, T=T, n=_log(rng, 2, min(128, T // 32)), H=H, d=d, dtype=dtype, lens=rng.randint(1, 10 ** 6))
    if kind == "layer":
        B = rng.randint(1, 4)
        return dict(kind=kind, B=B, T=_log(rng, 64, most // 2 // (B * H)), H=H, d=d, dtype=dtype)
    B = rng.randint(1, 4)
    return dict(kind=kind, B=B, T=_log(rng, 64, most // (B * H)), H=H, d=d, dtype=dtype, keep=rng.random() < 0.6,
                eta=rng.random() < 0.5, segment=rng.random() < 0.3)


def _offsets(case):
    """Cumulative offsets of n sequences of log-normal lengths, at least one token each, T tokens together."""
    T, n = case["T"], case["n"]
    rnd = random.Random(case["lens"])
    w = [rnd.lognormvariate(0.0, 0.8) for _ in range(n)]
    total, acc, cu = sum(w), 0.0, [0]
    for i in range(n):
        acc += w[i]
        cu.append(min(max(cu[-1] + 1, int(round(acc / total * T))), T - (n - 1 - i)))
    cu[-1] = T
    return cu


class _Inputs:
    """Random tensors on the GPU from one seed, with the distributions of the path."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def normal(self, *shape):
        return torch.randn(shape, device="cuda", generator=self.g)

    def values(self, *shape):
        return self.normal(*shape).to(self.dt)

    def unit(self, *shape):
        x = self.normal(*shape)
        return (x / x.norm(dim=-1, keepdim=True)).to(self.dt)

    def tokens(self, B, T, H, d):
        return dict(q=self.unit(B, T, H, d), k=self.unit(B, T, H, d), v=self.values(B, T, H, d),
                    beta=torch.sigmoid(self.normal(B, T, H)), alpha=torch.sigmoid(self.normal(B, T, H) + 3.0),
                    mu=torch.sigmoid(self.normal(B, T, H) + 2.0).clamp_(min=math.exp(-1.0)))

    def eta(self, B, T, H):
        return torch.tanh(self.normal(B, T, H)) + 1.0


def prepare(case, seed):
    kind, H, d, T = case["kind"], case["H"], case["d"], case["T"]
    B = case.get("B", 1)
    r = _Inputs(seed, case["dtype"])
    s = {"kind": kind, "scale": d ** -0.5}
    if kind == "layer":
        for name in ("x_q", "x_k", "x_v", "g", "dy"):
            s[name] = r.values(B, T, H, d)
        for name in ("x_alpha", "x_mu", "x_beta", "x_eta"):
            s[name] = r.normal(B, T, H)
        s["d"] = 0.3 * torch.sigmoid(r.normal(H))
        s["w"] = 1.0 + 0.1 * r.normal(d)
        # decay rates and biases: alpha around 0.95, mu around 0.85 at the typical token
        s["gates"] = (torch.exp(0.2 * r.normal(H)) * 0.5, r.normal(H) * 0.3 - 2.0, torch.exp(0.2 * r.normal(H)) * 0.5,
                      r.normal(H) * 0.3 - 1.0)
        s["f"], s["b"] = {}, {}
        return s
    s.update(r.tokens(B, T, H, d))
    if kind == "decode":
        s["S"], s["M"], s["o"] = 0.3 * r.normal(B, H, d, d), 0.1 * r.normal(B, H, d, d), None
    elif kind == "prefill":
        s["f"] = {}
    elif kind == "train":
        s["keep"] = case["keep"]
        s["eta"] = r.eta(B, T, H) if case["eta"] else None
        s["dO"] = r.values(B, T, H, d)
        seg = case["segment"]
        s["S0"], s["M0"] = (0.3 * r.normal(B, H, d, d), 0.1 * r.normal(B, H, d, d)) if seg else (None, None)
        s["dS"], s["dM"] = (0.1 * r.normal(B, H, d, d), 0.1 * r.normal(B, H, d, d)) if seg else (None, None)
        s["f"], s["b"] = {}, {}
    else:
        s["cu"] = _offsets(case)
        if kind == "packed_train":
            s["dO"] = r.values(B, T, H, d)
        else:
            n, carry = case["n"], case["carry"]
            s["S0"], s["M0"] = (0.3 * r.normal(n, H, d, d), 0.1 * r.normal(n, H, d, d)) if carry else (None, None)
    return s


def _decode(s, x):
    s["o"] = binding.mdn_recurrent_step(*x, s["S"], s["M"], scale=s["scale"], out=s["o"])
    return {"o": s["o"], "S": s["S"], "M": s["M"]}


def _prefill(s, x):
    s["f"] = binding.mdn_chunk_fwd(*x, scale=s["scale"], workspace=s["f"].get("workspace"), out=s["f"])
    return {k: s["f"][k] for k in ("o", "S", "M")}


def _train(s, x):
    keep = s["keep"]
    f = s["f"] = binding.mdn_chunk_fwd(*x, eta=s["eta"], S0=s["S0"], M0=s["M0"], scale=s["scale"], save_vt=True,
                                       save_states=keep, save_operands=keep, workspace=s["f"].get("workspace"), out=s["f"])
    b = s["b"] = binding.mdn_chunk_bwd(*x, f["vt"], s["dO"], eta=s["eta"], S0=s["S0"], M0=s["M0"], states=f["states"],
                                       operands=f["operands"], dS_final=s["dS"], dM_final=s["dM"], scale=s["scale"],
                                       want_deta=s["eta"] is not None, workspace=s["b"].get("workspace"), out=s["b"])
    out = {k: f[k] for k in ("o", "S", "M")}
    out.update((k, b[k]) for k in ("dq", "dk", "dv", "dbeta", "dalpha", "dmu", "deta", "dS0", "dM0"))
    return out


def _packed_prefill(s, x):
    f = binding.mdn_chunk_fwd_varlen(*x, s["cu"], S0=s["S0"], M0=s["M0"], scale=s["scale"])
    return {k: f[k] for k in ("o", "S", "M")}


def _packed_train(s, x):
    f = binding.mdn_chunk_fwd_varlen(*x, s["cu"], scale=s["scale"], save_vt=True, want_states=False)
    b = binding.mdn_chunk_bwd_varlen(*x, f["vt"], s["dO"], s["cu"], scale=s["scale"], want_state_grads=False)
    return {"o": f["o"], **{k: b[k] for k in ("dq", "dk", "dv", "dbeta", "dalpha", "dmu")}}


def _layer(s):
    xs = tuple(s[k] for k in ("x_alpha", "x_mu", "x_beta", "x_eta"))
    gate = binding.mdn_gates_fwd(*xs, *s["gates"], 0.5, 4.0)
    n = binding.mdn_frontend_fwd(s["x_q"], s["x_k"], s["x_v"], s["d"])
    x = (n["q"], n["k"], n["v"], gate["beta"], gate["alpha"], gate["mu"])
    f = s["f"] = binding.mdn_chunk_fwd(*x, eta=gate["eta"], scale=s["scale"], save_vt=True, save_states=True,
                                       save_operands=True, output_final_state=False, workspace=s["f"].get("workspace"),
                                       out=s["f"])
    y = binding.mdn_epilogue_fwd(f["o"], s["g"], s["w"])
    e = binding.mdn_epilogue_bwd(f["o"], s["g"], s["w"], s["dy"])
    b = s["b"] = binding.mdn_chunk_bwd(*x, f["vt"], e["do"], eta=gate["eta"], states=f["states"], operands=f["operands"],
                                       scale=s["scale"], want_deta=True, want_dstates=False,
                                       workspace=s["b"].get("workspace"), out=s["b"])
    fb = binding.mdn_frontend_bwd(s["x_q"], s["x_k"], s["x_v"], s["d"], b["dq"], b["dk"], b["dv"])
    gb = binding.mdn_gates_bwd(*xs, *s["gates"], 0.5, 4.0, b["dalpha"], b["dbeta"], b["dmu"], b["deta"])
    return {"y": y, "dg": e["dg"], "dw": e["dw"], **fb, **gb}


def run(state):
    if state["kind"] == "layer":
        return _layer(state)
    x = tuple(state[k] for k in NAMES)
    return {"decode": _decode, "prefill": _prefill, "train": _train, "packed_prefill": _packed_prefill,
            "packed_train": _packed_train}[state["kind"]](state, x)


def work(case):
    """Bytes: every tensor of the call once (what passes between forward and backward is not counted).  Operations: per
    token and head, the chunkwise algorithm at C = 64 (forward 12 d^2 + 10 C d + 2/3 C^2, backward 24 d^2 + 16 C d; states
    and chunk-local operands formed once), for decoding the recurrence itself (10 d^2)."""
    kind, H, d, T, B = case["kind"], case["H"], case["d"], case["T"], case.get("B", 1)
    es, C = (2 if case["dtype"] == "bf16" else 4), 64
    n = B * T * H
    row, state = n * d * es, 2 * H * d * d * 4
    fwd, bwd = n * (12 * d * d + 10 * C * d + 2 * C * C // 3), n * (24 * d * d + 16 * C * d)
    if kind == "decode":
        return {"bytes": 4 * row + 12 * n + 2 * B * state, "flops": 10 * d * d * n}
    if kind == "prefill":
        return {"bytes": 4 * row + 12 * n + B * state, "flops": fwd}
    if kind == "packed_prefill":
        return {"bytes": 4 * row + 12 * n + case["n"] * state * (2 if case["carry"] else 1), "flops": fwd}
    if kind == "packed_train":
        return {"bytes": 8 * row + 24 * n, "flops": fwd + bwd}
    if kind == "layer":
        # x_q, x_k, x_v, g, dy in; y, dx_q, dx_k, dx_v, dg out; four projections in, their gradients out
        return {"bytes": 10 * row + 32 * n, "flops": fwd + bwd}
    gates = (32 if case["eta"] else 24) * n
    return {"bytes": 8 * row + gates + B * state * (4 if case["segment"] else 2), "flops": fwd + bwd}


def tolerance(case):
    """Relative 2-norm error between two correct implementations.  32-bit storage: fp32 sums in another order.  16-bit
    storage: decoding rounds its outputs only (2^-8 / sqrt(3)); the chunkwise path also rounds what it hands from product
    to product."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 3e-3} if case["kind"] == "decode" else {"rel": 1e-2}

"""Performance cases of the framework: what is run, on which inputs, and what it cannot do without.

A case is one pass through the public entry points (paper_2407_12117_amd.binding), called as a training
program calls them.  Kinds:

  train       attention forward and backward of one layer, outputs allocated by the call
  fwd, bwd    one direction alone (evaluation and prefill; a backward whose forward ran earlier)
  static      forward and backward into buffers the caller keeps, without a workspace
              (memo_attn_bwd_static: serving loops, code under graph capture)
  packed      train on q, k, v that are slices of one [B, S, 3, H, d] projection output
  recompute   LayerNorm and the q, k, v projection of the dropped token rows [k, S)
  step        a layer's step with the token-wise swap of a saved activation beside it: swap-out under the
              forward, swap-in under the backward

Head counts are one GPU's share at tensor-parallel degree 8 of the 32- and 40-head models the workloads
in synth.CONFIGS are taken from (H = 4 and 5, h = 4096 and 5120); the small ones are those of the tests.
"""
import math

import torch

from paper_2407_12117_amd import binding as mb
from paper_2407_12117_amd import synth

_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
_LN_EPS = 1e-5


def _attn(name, kind, dtype, B, S, H, d):
    return dict(name=name, kind=kind, dtype=dtype, B=B, S=S, H=H, d=d)


def _recompute(name, S, h, N, alpha, bias):
    return dict(name=name, kind="recompute", dtype="bf16", S=S, h=h, N=N, alpha=alpha, bias=bias)


def listed():
    return [
        # the fp32 workload C1: the full-precision check of a short sequence, a few launches long
        _attn("f32_train_1k", "train", "f32", 1, 1024, 1, 64),
        # full precision at the head dim of the bf16 path, ragged, long enough to be arithmetic-bound
        _attn("f32_train_3000", "train", "f32", 1, 3000, 4, 128),
        # the smallest call in use: short prompts in a loop, everything preallocated; latency counts
        _attn("bf16_static_640", "static", "bf16", 1, 640, 2, 128),
        # short training sequences in a batch, ragged
        _attn("bf16_train_2x2000", "train", "bf16", 2, 2000, 3, 128),
        # forward only at an ordinary context length (evaluation, prefill)
        _attn("bf16_fwd_8k", "fwd", "bf16", 1, 8192, 4, 128),
        # ordinary context length, ragged, q k v in the packed layout a fused projection writes
        _attn("bf16_packed_16461", "packed", "bf16", 1, 16461, 4, 128),
        # C2: the shortest workload of the swap, where the copies are longer than the attention
        dict(name="step_32k", kind="step", dtype="bf16", B=1, S=32768, H=4, d=128, act_cols=4096, alpha=0.75),
        # a sequence length between the powers of two, head count of the 40-head model
        _attn("bf16_train_50000", "train", "bf16", 1, 50000, 5, 128),
        # C4: the backward of the 256K-token workload
        _attn("bf16_bwd_256k", "bwd", "bf16", 1, 262144, 5, 128),
        # C5: the forward of the 1M-token workload
        _attn("bf16_fwd_1m", "fwd", "bf16", 1, 1048576, 4, 128),
        # recomputation of the rows that the alpha of the 1M-token workload drops, at 256K tokens
        _recompute("recompute_256k", 262144, 4096, 1536, 0.47, True),
        # the same at a short length: a few thousand rows of the 40-head model's shapes, ragged
        _recompute("recompute_4k", 4100, 5120, 1920, 0.25, True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f32", "static", "train", "train", "fwd", "bwd", "packed", "step", "recompute", "recompute"])
    if kind == "f32":
        c = _attn("", rng.choice(["train", "fwd", "bwd"]), "f32", rng.randint(1, 2), _log_uniform(rng, 300, 5000),
                  rng.randint(1, 4), rng.choice([64, 128]))
    elif kind == "static":
        c = _attn("", kind, "bf16", rng.randint(1, 2), _log_uniform(rng, 200, 4000), rng.randint(1, 4), 128)
    elif kind == "train":
        c = _attn("", kind, "bf16", rng.randint(1, 2), _log_uniform(rng, 600, 100000), rng.randint(1, 5), 128)
    elif kind == "fwd":
        c = _attn("", kind, "bf16", 1, _log_uniform(rng, 2000, 400000), rng.choice([2, 4, 5]), 128)
    elif kind == "bwd":
        c = _attn("", kind, "bf16", 1, _log_uniform(rng, 2000, 200000), rng.choice([2, 4, 5]), 128)
    elif kind == "packed":
        c = _attn("", kind, "bf16", rng.randint(1, 2), _log_uniform(rng, 1000, 50000), rng.choice([4, 5]), 128)
    elif kind == "step":
        H = rng.choice([4, 5])
        c = dict(kind=kind, dtype="bf16", B=1, S=_log_uniform(rng, 16000, 65536), H=H, d=128, act_cols=1024 * H,
                 alpha=rng.choice([0.125, 0.25, 0.5, 0.75, 1.0]))
    else:
        h, N = rng.choice([(4096, 1536), (5120, 1920), (1024, 384)])
        c = _recompute("", _log_uniform(rng, 300, 262144), h, N, rng.choice([0.0, 0.125, 0.25, 0.47, 0.75]),
                       rng.random() < 0.7)
    c.pop("name", None)
    return c


def _recompute_rows(case):
    return mb.memo_split_tokens(case["S"], case["alpha"]), case["S"]


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind}
    if kind == "recompute":
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed))
        S, h, N = case["S"], case["h"], case["N"]

        def normal(*shape):
            return torch.randn(shape, generator=g, dtype=torch.float32, device="cuda")

        st["x"] = torch.empty((S, h), dtype=torch.bfloat16, device="cuda")
        for r in range(0, S, 65536):      # in pieces: the fp32 draw of a long sequence need not exist whole
            n = min(65536, S - r)
            st["x"][r:r + n] = normal(n, h)
        st["gamma"] = (1.0 + 0.1 * normal(h)).to(torch.bfloat16)
        st["beta"] = (0.1 * normal(h)).to(torch.bfloat16)
        st["w"] = (normal(N, h) / math.sqrt(h)).to(torch.bfloat16)
        st["bias"] = (0.1 * normal(N)).to(torch.bfloat16) if case["bias"] else None
        # rows [0, k) are the ones that came back from the host
        st["norm"] = torch.zeros_like(st["x"])
        st["qkv"] = torch.zeros((S, N), dtype=torch.bfloat16, device="cuda")
        st["rows"] = _recompute_rows(case)
        return st

    B, S, H, d = case["B"], case["S"], case["H"], case["d"]
    st["scale"] = synth.default_scale(d)
    q, k, v, g = synth.attn_inputs(B, S, H, d, case["dtype"], seed, device="cuda")
    if kind == "packed":
        qkv = torch.stack((q, k, v), dim=2)
        q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
        d_o = torch.zeros_like(qkv)
        d_o[:, :, 0] = g
        g = d_o[:, :, 0]
        st["o_buf"], st["grads"] = torch.zeros_like(qkv), torch.zeros_like(qkv)
    st.update(q=q, k=k, v=v, g=g)
    if kind == "bwd":
        st["o"], st["lse"] = mb.memo_attn_fwd(q, k, v, st["scale"])
    elif kind == "static":
        st["o"], st["dq"], st["dk"], st["dv"] = (torch.zeros_like(q) for _ in range(4))
        st["lse"] = torch.zeros((B, H, S), dtype=torch.float32, device="cuda")
    elif kind == "step":
        st["alpha"] = case["alpha"]
        st["act"] = synth.activation(S, case["act_cols"] * 2, seed, device="cuda")
        st["back"] = torch.zeros_like(st["act"])
        plan = mb.memo_swap_plan_make(S, case["act_cols"] * 2, case["alpha"])
        st["host"] = torch.zeros(max(1, plan["bytes_swapped"]), dtype=torch.uint8, pin_memory=True)
        st["offload"], st["prefetch"] = torch.cuda.Stream(), torch.cuda.Stream()
        for name in ("ready", "out_done", "fwd_done", "in_done"):
            st[name] = torch.cuda.Event()
    return st


def run(st):
    kind = st["kind"]
    if kind == "recompute":
        mb.memo_layernorm_rows(st["x"], st["gamma"], st["beta"], _LN_EPS, y=st["norm"], rows=st["rows"])
        mb.memo_linear_rows(st["norm"], st["w"], st["bias"], out=st["qkv"], rows=st["rows"])
        return st["norm"], st["qkv"]
    q, k, v, g, scale = st["q"], st["k"], st["v"], st["g"], st["scale"]
    if kind == "fwd":
        return mb.memo_attn_fwd(q, k, v, scale)
    if kind == "bwd":
        return mb.memo_attn_bwd(q, k, v, st["o"], st["lse"], g, scale)
    if kind == "train":
        o, lse = mb.memo_attn_fwd(q, k, v, scale)
        return (o, lse) + mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    if kind == "static":
        o, lse = mb.memo_attn_fwd(q, k, v, scale, o=st["o"], lse=st["lse"])
        return (o, lse) + mb.memo_attn_bwd_static(q, k, v, o, lse, g, scale, st["dq"], st["dk"], st["dv"])
    if kind == "packed":
        o, lse = mb.memo_attn_fwd(q, k, v, scale, o=st["o_buf"][:, :, 0])
        gr = st["grads"]
        mb.memo_attn_bwd(q, k, v, o, lse, g, scale, dq=gr[:, :, 0], dk=gr[:, :, 1], dv=gr[:, :, 2])
        return o, lse, gr
    # step: the activation leaves under the forward and comes back under the backward
    here = torch.cuda.current_stream()
    st["ready"].record(here)
    mb.memo_swap_out(st["act"], st["alpha"], st["host"], st["offload"], wait_event=st["ready"], done_event=st["out_done"])
    o, lse = mb.memo_attn_fwd(q, k, v, scale)
    st["fwd_done"].record(here)
    st["prefetch"].wait_event(st["out_done"])
    mb.memo_swap_in(st["back"], st["alpha"], st["host"], st["prefetch"], wait_event=st["fwd_done"], done_event=st["in_done"])
    grads = mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    here.wait_event(st["in_done"])
    return (o, lse) + grads + (st["back"], st["host"])


def work(case):
    kind = case["kind"]
    if kind == "recompute":
        k, S = _recompute_rows(case)
        n, h, N = S - k, case["h"], case["N"]
        # x in, norm out, q k v out, weights; the projection's flops
        return {"bytes": 2 * (2 * n * h + n * N + N * h + 2 * h + (N if case["bias"] else 0)), "flops": 2 * n * h * N}
    B, S, H, d = case["B"], case["S"], case["H"], case["d"]
    tensor = B * S * H * d * _DTYPES[case["dtype"]].itemsize
    stat = B * H * S * 4
    pairs = B * H * (S * (S + 1) // 2)            # visible (query, key) pairs; 2 d flops per pair and contraction
    fwd = {"bytes": 4 * tensor + stat, "flops": 2 * 2 * d * pairs}
    bwd = {"bytes": 8 * tensor + stat, "flops": 5 * 2 * d * pairs}
    if kind == "fwd":
        return fwd
    if kind == "bwd":
        return bwd
    # the forward's outputs are the backward's inputs; q, k, v are read once
    both = {"bytes": 8 * tensor + stat, "flops": fwd["flops"] + bwd["flops"]}
    if kind == "step":
        both["bytes"] += 4 * mb.memo_split_tokens(S, case["alpha"]) * case["act_cols"] * 2   # device and host side of both copies
    return both


def tolerance(case):
    # About four times the relative 2-norm error against the same operations in 64 bits: bf16 attention 2.5e-3
    # (gradients; 16461 tokens as 640), fp32 attention 1.3e-6 (dK at 3000 tokens, growing with the length),
    # LayerNorm 1.7e-3 and the projection behind it 2.3e-3.  Bytes that are swapped come back as they were.
    if case["kind"] == "recompute":
        return {"rel": 9e-3}
    if case["dtype"] == "f32":
        return {"rel": 6e-6}
    return {"rel": 1e-2}

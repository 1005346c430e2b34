"""The calls a program makes to this library, as cases that can be timed and compared.

A case is one call (or, where token features come in, the routing map and the call behind it)
through the public entry points, at one size, data type and set of options:

  prefill   swimba_mixer_fwd on a batch of sequences (prompt processing, evaluation, the forward of
            training), from a zero or a given initial state, with the final state handed back
  features  swimba_router_linear + swimba_mixer_fwd_proj: token features to y, B and C of the selected
            experts projected inside the call
  xe        swimba_router_linear + swimba_mixer_fwd_xe_proj: the same with one projected input stream
            per expert
  decode    swimba_step: one token per sequence, the state updated in place
  multi     swimba_step_multi: a few tokens per sequence in one call (speculative decoding), the state
            updated in place

Values are drawn as in paper_2603_06938_amd/synth.py: x and the logits standard normal, B and C
N(0, 1/N), dt = softplus(normal + bias) around step sizes log-uniform in [1e-3, 1e-1], A log-uniform
in [-16, -1], D = 1, carried states N(0, 0.1).
"""
import math

import torch

from paper_2603_06938_amd import binding as sw

DEVICE = "cuda:0"
IO = {"f32": torch.float32, "bf16": torch.bfloat16}


def _prefill(name, B, L, H, P, N, G, E, k, Q, io, h0=False, skip=True):
    return {"name": name, "kind": "prefill", "batch": B, "seqlen": L, "nheads": H, "headdim": P, "dstate": N,
            "ngroups": G, "nexperts": E, "top_k": k, "chunk": Q, "io": io, "h0": h0, "skip": skip, "d_model": 0}


def _case(kind, name, B, L, H, P, N, G, E, k, Q, io, d_model=0):
    c = _prefill(name, B, L, H, P, N, G, E, k, Q, io)
    c.update(kind=kind, d_model=d_model, h0=kind in ("decode", "multi"))
    return c


def listed():
    return [
        # unit-sized fp32 problem: what a check of the mathematics runs; nothing but latency
        _prefill("prefill_tiny_f32", 1, 256, 4, 16, 16, 1, 4, 2, 64, "f32"),
        # one short prompt of one user in the 130M-shaped layer: time to first token
        _prefill("prefill_one_prompt", 1, 150, 24, 64, 128, 1, 8, 2, 256, "bf16"),
        # a batch of prompts of odd length continued from earlier states (chunked prefill, next turn of a chat)
        _prefill("prefill_ragged_h0", 5, 1237, 32, 64, 128, 1, 8, 2, 256, "bf16", h0=True),
        # the 130M-shaped layer at its training length
        _prefill("prefill_130m", 8, 2048, 24, 64, 128, 1, 8, 2, 256, "bf16"),
        # the 370M-shaped layer
        _prefill("prefill_370m", 8, 4096, 32, 64, 128, 1, 8, 2, 256, "bf16"),
        # long documents, B/C in 8 groups, 16 experts
        _prefill("prefill_long", 2, 16384, 64, 64, 128, 8, 16, 2, 256, "bf16"),
        # the 130M-shaped layer in full precision (reference runs, numerics-sensitive evaluation)
        _prefill("prefill_130m_f32", 2, 2048, 24, 64, 128, 1, 8, 2, 256, "f32"),
        # token features to y in one call: the layer as a model calls it
        _case("features", "features_130m", 8, 2048, 24, 64, 128, 1, 8, 2, 256, "bf16", d_model=768),
        # the same with an input stream of its own for each expert
        _case("xe", "features_xe_130m", 4, 2048, 24, 64, 128, 1, 8, 2, 256, "bf16", d_model=768),
        # one user's decode step: launches and host path
        _case("decode", "decode_one", 1, 1, 24, 64, 128, 1, 8, 2, 0, "bf16"),
        # a full serving batch: the state streams through memory once
        _case("decode", "decode_batch", 64, 1, 64, 64, 128, 1, 8, 2, 0, "bf16"),
        # speculative decoding: four drafted tokens verified per call
        _case("multi", "decode_multi", 16, 4, 64, 64, 128, 1, 8, 2, 0, "bf16"),
    ]


# Ranges behind the listed cases.  A drawn prefill has at most as many tokens x heads as its largest listed
# relative of the same data type and at most as many tokens x groups as the long documents, so no drawn case
# costs more than the largest listed one.
TOKEN_HEADS = {"bf16": 8 * 4096 * 32, "f32": 2 * 2048 * 24, "features": 8 * 2048 * 24, "xe": 4 * 2048 * 24}
TOKEN_GROUPS = 2 * 16384 * 8


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill"] * 5 + ["prefill_f32"] * 2 + ["features", "xe"] + ["decode"] * 2 + ["multi"])
    io = "f32" if kind == "prefill_f32" else "bf16"
    H = rng.choice([8, 16, 24, 24, 32, 32, 48, 64])
    # the layer's sizes: 64 channels and 128 states per head as the named layers have, and their smaller relatives
    P, N = rng.choice([(64, 128)] * 5 + [(64, 64), (32, 128), (64, 16)])
    G = rng.choice([1, 1, 1, 2, 4, 8])
    E = rng.choice([4, 8, 8, 16])
    k = rng.choice([1, 2, 2, 2])
    if kind in ("decode", "multi"):
        B = _log_int(rng, 1, 96)
        L = 1 if kind == "decode" else rng.randint(2, 8)
        return {q: v for q, v in _case(kind, "", B, L, H, P, N, G, E, k, 0, io).items() if q != "name"}
    most = TOKEN_HEADS[io if kind.startswith("prefill") else kind]
    Q = rng.choice([64, 128, 256, 256, 256, 256])
    tokens = _log_int(rng, 100, min(most // H, TOKEN_GROUPS // G))
    B = min(_log_int(rng, 1, 16), max(1, tokens // 64))
    L = max(1, min(tokens // B, 16384))
    if rng.random() < 0.5 and L > Q:
        L = L // Q * Q                                  # padded batches: whole chunks
    if kind.startswith("prefill"):
        c = _prefill("", B, L, H, P, N, G, E, k, Q, io, h0=rng.random() < 0.4, skip=rng.random() < 0.8)
    else:
        c = _case(kind, "", B, L, H, 64, rng.choice([64, 128, 128]), 1, E, k, Q, io, d_model=rng.choice([512, 768, 1024]))
    return {q: v for q, v in c.items() if q != "name"}


def prepare(case, seed):
    c = dict(case)
    io = IO[c["io"]]
    B, L, H, P, N, G, E, k = (c[q] for q in ("batch", "seqlen", "nheads", "headdim", "dstate", "ngroups", "nexperts", "top_k"))
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)

    def normal(shape, scale=1.0, dtype=io):
        t = torch.randn(shape, generator=gen, device=DEVICE, dtype=dtype)
        return t if scale == 1.0 else t.mul_(scale)

    lead = (B,) if c["kind"] == "decode" else (B, L)
    st = {"case": c}
    dt0 = torch.exp(math.log(1e-3) + math.log(1e2) * torch.rand(H, generator=gen, device=DEVICE))
    z = torch.randn(lead + (H,), generator=gen, device=DEVICE)
    st["dt"] = torch.nn.functional.softplus(z + torch.log(torch.expm1(dt0))).to(io)
    st["A"] = -torch.exp(math.log(16.0) * torch.rand(H, generator=gen, device=DEVICE))
    st["D"] = torch.ones(H, device=DEVICE) if c["skip"] else None
    if c["kind"] != "xe":
        st["x"] = normal(lead + (H, P))
    if c["d_model"]:
        Dm = c["d_model"]
        st["u"] = normal((B, L, Dm))
        st["W_g"] = normal((E, Dm), Dm ** -0.5)
        st["W_B"] = normal((E, G, N, Dm), (Dm * N) ** -0.5)
        st["W_C"] = normal((E, G, N, Dm), (Dm * N) ** -0.5)
        if c["kind"] == "xe":
            st["W_X"] = normal((E, H, P, Dm), Dm ** -0.5)
    else:
        st["B"] = normal(lead + (E, G, N), N ** -0.5)
        st["C"] = normal(lead + (E, G, N), N ** -0.5)
        st["logits"] = normal(lead + (E,))
    st["h"] = normal((B, H, P, N), 0.1, torch.float32) if c["h0"] else None
    # the scratch a program allocates once per shape
    dims = sw.make_dims(B, L, H, P, N, G, E, k, c["chunk"], io)
    size = {"prefill": lambda: sw.swimba_mixer_workspace_bytes(dims),
            "features": lambda: sw.swimba_mixer_proj_workspace_bytes(dims, c["d_model"]),
            "xe": lambda: sw.swimba_mixer_xe_proj_workspace_bytes(dims, c["d_model"]),
            "decode": lambda: sw.swimba_step_workspace_bytes(dims),
            "multi": lambda: sw.swimba_step_multi_workspace_bytes(dims)}[c["kind"]]()
    st["ws"] = torch.empty(size, dtype=torch.uint8, device=DEVICE)
    return st


def run(state):
    s, c = state, state["case"]
    k, Q = c["top_k"], c["chunk"]
    if c["kind"] == "prefill":
        out = sw.swimba_mixer_fwd(s["x"], s["dt"], s["A"], s["D"], s["B"], s["C"], s["logits"], k, Q, s["h"],
                                  workspace=s["ws"])
        return {"y": out.y, "h_final": out.h_final}
    if c["kind"] == "features":
        logits = sw.swimba_router_linear(s["u"], s["W_g"])
        out = sw.swimba_mixer_fwd_proj(s["u"], s["W_B"], s["W_C"], s["x"], s["dt"], s["A"], s["D"], logits, k, Q,
                                       workspace=s["ws"])
        return {"y": out.y, "h_final": out.h_final}
    if c["kind"] == "xe":
        logits = sw.swimba_router_linear(s["u"], s["W_g"])
        out = sw.swimba_mixer_fwd_xe_proj(s["u"], s["W_B"], s["W_C"], s["W_X"], s["dt"], s["A"], s["D"], logits, k, Q,
                                          workspace=s["ws"])
        return {"y": out.y, "h_final": out.h_final}
    step = sw.swimba_step if c["kind"] == "decode" else sw.swimba_step_multi
    out = step(s["h"], s["x"], s["dt"], s["A"], s["D"], s["B"], s["C"], s["logits"], k, workspace=s["ws"])
    return {"y": out.y, "state": out.state}


def work(case):
    B, L, H, P, N, G, E, k, Dm = (case[q] for q in ("batch", "seqlen", "nheads", "headdim", "dstate", "ngroups",
                                                    "nexperts", "top_k", "d_model"))
    e = 2 if case["io"] == "bf16" else 4
    T = B * L
    # the recurrence itself: decay, injection and readout of every state element, once per token
    flops = 5.0 * T * H * P * N
    nbytes = T * H * (P + 1) * e                        # y, dt
    if Dm:
        cols = 2 * G * N + (H * P if case["kind"] == "xe" else 0)
        nbytes += T * Dm * e + E * (cols + 1) * Dm * e  # features, weights
        flops += 2.0 * T * Dm * (k * cols + E)
    else:
        nbytes += T * (E + 2 * k * G * N) * e           # logits, B and C rows of the selected experts
        flops += 4.0 * T * k * G * N
    if case["kind"] != "xe":
        nbytes += T * H * P * e                         # x
    nbytes += B * H * P * N * 4 * (2 if case["h0"] else 1)   # states in (where given) and out
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    if case["io"] == "f32":
        return {"rel": 1e-5}                            # fp32 sums of up to a few hundred terms, exponentials of fp32 sums
    if case["kind"] in ("decode", "multi"):
        return {"rel": 4e-3}                            # fp32 arithmetic; y is rounded to bf16
    return {"rel": 1e-2}                                # bf16 operands, fp32 accumulation

"""The work this library is measured on: one layer's hybrid-attention operator as a serving or a training program calls it.

Five kinds of calls, each through the public entry points of `paper_2602_02180_amd.binding`:

  prefill   still_hybrid_attn_fwd over whole sequences
  decode    one still_hybrid_attn_decode_step behind a prefilled context (a step that does not route a chunk, so that it
            can be repeated on the same state: it rewrites the new token's ring slot and score and its output)
  generate  a prompt and its first tokens: prefill of a right-padded batch with the decode state exported, then
            still_hybrid_attn_decode_step_at steps at per-sequence positions, some of which route a chunk
  train     still_hybrid_attn_fwd + still_hybrid_attn_bwd
  transfer  the attention-transfer stage: still_hybrid_attn_fwd, still_attention_map, still_attention_map_bwd

Inputs have the distributions of `synth.make_inputs` (per-channel log-normal scales; 1 % heavy-hitter keys where the
case says so) and are drawn on the GPU from the seed alone.  Workspaces, states, outputs and the parameter block are what
a program keeps between calls, so `prepare` makes them.
"""
import math

import torch

from paper_2602_02180_amd import binding as S

_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
EPS = 1e-6


def _case(name, kind, **kw):
    c = dict(kind=kind, B=1, N=1024, Hq=32, Hkv=8, d=128, C=128, W=128, lam=16, dtype="bf16", gate="none", bias=False,
             heavy=False, ragged=False, budget=0, shared=False, steps=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a two-head fp32 layer of 1024 tokens (the library's correctness configuration c1); latency
        # and the number of launches decide
        _case("prefill_tiny_f32", "prefill", N=1024, Hq=2, Hkv=2, d=64, C=64, W=64, dtype="f32"),
        # a batch of ordinary prompts on a 1B-shaped layer (configuration c2)
        _case("prefill_1b_4k", "prefill", B=4, N=4096, d=64, C=64, W=64),
        # ordinary long prompts on an 8B-shaped layer (c3)
        _case("prefill_8b_8k", "prefill", B=2, N=8192, C=64, W=128),
        # the long context the library's headline figure is quoted on (c4)
        _case("prefill_8b_32k", "prefill", N=32768, heavy=True),
        # a serving batch as it comes: right-padded prompts of odd lengths, a gate given as a pre-activation, biases
        _case("prefill_8b_ragged", "prefill", B=5, N=3001, gate="logit", bias=True, ragged=True),
        # decode at full batch behind a 32K context (c5), half a chunk into the generation
        _case("decode_8b_32k", "decode", B=64, N=32768 + 60, heavy=True),
        # one interactive sequence behind a 4K context: latency
        _case("decode_8b_single", "decode", B=1, N=4096 + 33),
        # a small-model batch whose retained rows are capped at 896, with gate and biases
        _case("decode_1b_budget", "decode", B=24, N=8192 + 21, d=64, C=64, W=64, budget=896, gate="given", bias=True),
        # a serving request: prompts of different lengths, then 24 tokens each at their own positions
        _case("generate_8b", "generate", B=8, N=2048, ragged=True, steps=24),
        # a training step at the training length of 1024 tokens (c6)
        _case("train_8b_1k", "train", B=16, N=1024, C=64, gate="given"),
        # a small training step of odd length on a 1B-shaped layer, gate activated inside, biases trained
        _case("train_1b_odd", "train", B=3, N=777, d=64, C=64, W=64, gate="logit", bias=True),
        # the attention-transfer stage at the training length
        _case("transfer_8b_1k", "transfer", B=4, N=1024, C=64, W=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: sizes spread over their logarithms, odd ones among them."""
    kind = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "generate", "train", "train", "transfer"])
    d = rng.choice([64, 128, 128])
    C = rng.choice([64, 128])
    c = _case(None, kind, d=d, C=C, W=rng.choice([64, 128]), lam=rng.choice([8, 16, 16, 32]),
              gate=rng.choice(["none", "given", "logit"]), bias=rng.random() < 0.3)
    Hq, Hkv = rng.choice([(32, 8), (32, 8), (16, 4), (8, 8)])
    c.update(Hq=Hq, Hkv=Hkv)
    if kind == "prefill":
        tokens = _log_int(rng, 1024, 32768)                  # of the whole batch
        c["B"] = rng.choice([1, 1, 2, 3, 4, 8])
        c["N"] = max(130, tokens // c["B"] + rng.randint(-40, 40))
        if tokens <= 4096 and rng.random() < 0.3:
            c["dtype"] = "f32"
        c["lam"] = min(c["lam"], 16) if c["N"] > 16384 else c["lam"]
        c["ragged"] = c["B"] > 1 and rng.random() < 0.5
        c["heavy"] = rng.random() < 0.3
        c["budget"] = rng.choice([0, 0, 0, 896])
        c["shared"] = rng.random() < 0.15
    elif kind == "decode":
        c["B"] = _log_int(rng, 1, 64)
        c["N"] = min(_log_int(rng, 300, 32768), 64 * 32768 // c["B"])
        c["N"] += 7 if c["N"] % C == 0 else 0                # (a step that routes could not be repeated)
        c["lam"] = min(c["lam"], 16)
        c["heavy"] = rng.random() < 0.3
        c["budget"] = rng.choice([0, 0, 896])
        c["shared"] = rng.random() < 0.2
    elif kind == "generate":
        c["B"], c["N"], c["steps"] = rng.randint(1, 12), _log_int(rng, 300, 2048), rng.randint(8, 32)
        c["ragged"] = True
    elif kind == "train":
        c["N"] = _log_int(rng, 200, 2048)
        c["B"] = rng.randint(1, max(1, min(16, 16384 // c["N"])))
        if d == 64 and c["B"] * c["N"] <= 2048 and rng.random() < 0.4:
            c["dtype"] = "f32"
    else:
        c["N"] = _log_int(rng, 200, 1024)
        c["B"] = rng.randint(1, 4)
        c["gate"] = "none"
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)


def _weights(case, gen):
    Hq, d, dt = case["Hq"], case["d"], _TORCH[case["dtype"]]
    w = {"Wq": (_normal(gen, Hq, d, d) / d ** 0.5).to(dt), "Wk": (_normal(gen, Hq, d, d) / d ** 0.5).to(dt),
         "bq": None, "bk": None}
    if case["bias"]:
        w["bq"], w["bk"] = (0.1 * _normal(gen, Hq, d)).to(dt), (0.1 * _normal(gen, Hq, d)).to(dt)
    scales = tuple(torch.exp(0.5 * _normal(gen, h, d)) for h in (case["Hq"], case["Hkv"], case["Hkv"]))
    return w, scales


def _gate(case, gen, *shape):
    if case["gate"] == "none":
        return None
    x = _normal(gen, *shape)
    return (torch.sigmoid(x) if case["gate"] == "given" else x).to(_TORCH[case["dtype"]])


def _qkv(case, gen, scales, B, N):
    dt = _TORCH[case["dtype"]]
    q, k, v = (_normal(gen, B, N, s.shape[0], case["d"]).mul_(s) for s in scales)
    if case["heavy"]:                                        # 1 % of the positions carry keys of eight times the norm
        pos = torch.rand(B, N, generator=gen, device="cuda").argsort(dim=1)[:, : max(1, N // 100)]
        for b in range(B):
            k[b, pos[b]] *= 8.0
    return q.to(dt), k.to(dt), v.to(dt)


def _base(case, B):
    return dict(B=B, Hq=case["Hq"], Hkv=case["Hkv"], d=case["d"], C=case["C"], W=case["W"], lam=case["lam"],
                scale=case["d"] ** -0.5, eps=EPS, dtype=case["dtype"], max_retained=case["budget"],
                shared_selection=int(case["shared"]), gate_activation=int(case["gate"] == "logit"))


def _bytes(n):
    return torch.zeros(max(int(n), 16), dtype=torch.uint8, device="cuda")


def _region(buf, off, n, dtype):
    size = torch.empty((), dtype=dtype).element_size()
    return buf[off: off + n * size].view(dtype)


def _lengths(case, gen):
    """Lengths of a right-padded batch: the longest fills the batch, the others are anything from half of it."""
    N, B = case["N"], case["B"]
    n = torch.randint(max(1, N // 2), N + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
    n[0] = N
    return n


def prepare(case, seed):
    return {"prefill": _prep_prefill, "decode": _prep_decode, "generate": _prep_generate, "train": _prep_train,
            "transfer": _prep_train}[case["kind"]](case, _gen(seed))


def _prep_prefill(case, gen):
    w, scales = _weights(case, gen)
    B, N = case["B"], case["N"]
    q, k, v = _qkv(case, gen, scales, B, N)
    g = _gate(case, gen, B, N, case["Hq"], case["d"])
    out = torch.zeros_like(q)
    sel = torch.full((B, case["Hq"], max(N // case["C"], 1), case["lam"]), -1, dtype=torch.int32, device="cuda")
    seq_len = _lengths(case, gen) if case["ragged"] else None
    p = S.make_params(N=N, q=q, k=k, v=v, out=out, g=g, seq_len=seq_len, **_base(case, B))
    return dict(case=case, p=p, q=q, k=k, v=v, g=g, out=out, sel=sel, ws=_bytes(S.still_fwd_workspace_bytes(p)), **w)


def _state_regions(case, L, B):
    """(offset, elements, type) of the regions of a decode state, the scratch region left out."""
    d, Hq, Hkv, dt = case["d"], case["Hq"], case["Hkv"], _TORCH[case["dtype"]]
    slices = Hkv if case["shared"] else Hq
    return {"S": (L.S, B * Hq * 2 * d * (d + 1), torch.float32), "kret": (L.kret, B * slices * L.cap * d, dt),
            "vret": (L.vret, B * slices * L.cap * d, dt), "sel": (L.sel, B * Hq * L.n_chunks * case["lam"], torch.int32),
            "kring": (L.kring, B * Hkv * L.R * d, dt), "vring": (L.vring, B * Hkv * L.R * d, dt),
            "score": (L.score, B * Hq * L.R, torch.float32)}


def _prep_decode(case, gen):
    """The state behind N tokens per sequence, prefilled a few sequences at a time."""
    w, scales = _weights(case, gen)
    B, N, Hq, Hkv, d = case["B"], case["N"], case["Hq"], case["Hkv"], case["d"]
    dt = _TORCH[case["dtype"]]
    cap = N + 256
    ps = S.make_params(N=1, max_tokens=cap, **_base(case, B))
    state = _bytes(S.still_state_bytes(ps))
    regions = _state_regions(case, S.still_state_layout(ps), B)
    per_call = max(1, min(B, 262144 // N))
    for b0 in range(0, B, per_call):
        n_b = min(per_call, B - b0)
        q, k, v = _qkv(case, gen, scales, n_b, N)
        out = torch.empty_like(q)
        p = S.make_params(N=N, max_tokens=cap, q=q, k=k, v=v, out=out, **_base(case, n_b))
        part = _bytes(S.still_state_bytes(p))
        S.still_hybrid_attn_fwd(p, q, k, v, None, w["Wq"], w["bq"], w["Wk"], w["bk"], out, state_out=part,
                                workspace=_bytes(S.still_fwd_workspace_bytes(p)))
        for name, (off, n, ty) in _state_regions(case, S.still_state_layout(p), n_b).items():
            dst = _region(state, regions[name][0], regions[name][1], ty)
            one = n // n_b
            dst[b0 * one: b0 * one + n] = _region(part, off, n, ty)
    q, k, v = (_normal(gen, B, s.shape[0], d).mul_(s).to(dt) for s in scales)
    return dict(case=case, p=ps, state=state, t=N, q=q, k=k, v=v, g=_gate(case, gen, B, Hq, d),
                out=torch.zeros(B, Hq, d, dtype=dt, device="cuda"),
                seen=[_region(state, *regions[n]) for n in ("score", "kring", "vring")], **w)


def _prep_generate(case, gen):
    w, scales = _weights(case, gen)
    B, N, Hq, Hkv, d, T = case["B"], case["N"], case["Hq"], case["Hkv"], case["d"], case["steps"]
    dt = _TORCH[case["dtype"]]
    q, k, v = _qkv(case, gen, scales, B, N)
    g = _gate(case, gen, B, N, Hq, d)
    seq_len = _lengths(case, gen)
    out = torch.zeros_like(q)
    p = S.make_params(N=N, q=q, k=k, v=v, out=out, g=g, seq_len=seq_len, max_tokens=N + T + 8, **_base(case, B))
    ps = S.make_params(N=1, max_tokens=N + T + 8, **_base(case, B))
    state = _bytes(S.still_state_bytes(p))
    regions = _state_regions(case, S.still_state_layout(ps), B)
    qt, kt, vt = (_normal(gen, T, B, s.shape[0], d).mul_(s).to(dt) for s in scales)
    return dict(case=case, p=p, ps=ps, q=q, k=k, v=v, g=g, out=out, seq_len=seq_len, pos=seq_len.clone(), state=state,
                qt=qt, kt=kt, vt=vt, gt=_gate(case, gen, T, B, Hq, d),
                outs=torch.zeros(T, B, Hq, d, dtype=dt, device="cuda"),
                ws=_bytes(S.still_fwd_workspace_bytes(p)), seen=[_region(state, *r) for r in regions.values()], **w)


def _prep_train(case, gen):
    w, scales = _weights(case, gen)
    B, N, Hq, d = case["B"], case["N"], case["Hq"], case["d"]
    q, k, v = _qkv(case, gen, scales, B, N)
    g = _gate(case, gen, B, N, Hq, d)
    out = torch.zeros_like(q)
    p = S.make_params(N=N, q=q, k=k, v=v, out=out, g=g, **_base(case, B))
    sel = torch.full((B, Hq, max(N // case["C"], 1), case["lam"]), -1, dtype=torch.int32, device="cuda")
    ws = _bytes(S.still_fwd_workspace_bytes(p))
    lse = _region(ws, S.still_fwd_workspace_layout(p).lse, B * Hq * N, torch.float32)
    f32 = dict(dtype=torch.float32, device="cuda")
    grads = {"dWq": torch.zeros(Hq, d, d, **f32), "dWk": torch.zeros(Hq, d, d, **f32),
             "dbq": torch.zeros(Hq, d, **f32) if case["bias"] else None,
             "dbk": torch.zeros(Hq, d, **f32) if case["bias"] else None}
    st = dict(case=case, p=p, q=q, k=k, v=v, g=g, out=out, sel=sel, ws=ws, lse=lse, grads=grads, **w)
    if case["kind"] == "train":
        st["dout"] = _normal(gen, *q.shape).to(q.dtype)
        grads.update(dq=torch.zeros_like(q), dk=torch.zeros_like(k), dv=torch.zeros_like(v),
                     dg=None if g is None else torch.zeros_like(g))
        st["bws"] = _bytes(S.still_bwd_workspace_bytes(p))
    else:
        st["map"] = torch.zeros(B, Hq, N, N, **f32)
        st["dmap"] = _normal(gen, B, Hq, N, N).tril_()
        st["bws"] = _bytes(S.still_attention_map_bwd_workspace_bytes(p))
    return st


# ------------------------------------------------------------------ one pass

def run(state):
    return {"prefill": _run_prefill, "decode": _run_decode, "generate": _run_generate, "train": _run_train,
            "transfer": _run_transfer}[state["case"]["kind"]](state)


def _run_prefill(s):
    S.still_hybrid_attn_fwd(s["p"], s["q"], s["k"], s["v"], s["g"], s["Wq"], s["bq"], s["Wk"], s["bk"], s["out"],
                            sel_idx=s["sel"], workspace=s["ws"])
    if s["case"]["ragged"]:                                  # (the lists of the padding are unspecified)
        return s["out"]
    return [s["out"], s["sel"]]


def _run_decode(s):
    S.still_hybrid_attn_decode_step(s["p"], s["state"], s["t"], s["q"], s["k"], s["v"], s["g"], s["Wq"], s["bq"],
                                    s["Wk"], s["bk"], s["out"])
    return [s["out"]] + s["seen"]


def _run_generate(s):
    S.still_hybrid_attn_fwd(s["p"], s["q"], s["k"], s["v"], s["g"], s["Wq"], s["bq"], s["Wk"], s["bk"], s["out"],
                            state_out=s["state"], workspace=s["ws"])
    pos, N, gt = s["pos"], s["case"]["N"], s["gt"]
    pos.copy_(s["seq_len"])
    for i in range(s["case"]["steps"]):
        S.still_hybrid_attn_decode_step_at(s["ps"], s["state"], pos, N + i, s["qt"][i], s["kt"][i], s["vt"][i],
                                           None if gt is None else gt[i], s["Wq"], s["bq"], s["Wk"], s["bk"], s["outs"][i])
        pos.add_(1)
    return [s["out"], s["outs"]] + s["seen"]


def _run_train(s):
    g = s["grads"]
    S.still_hybrid_attn_fwd(s["p"], s["q"], s["k"], s["v"], s["g"], s["Wq"], s["bq"], s["Wk"], s["bk"], s["out"],
                            sel_idx=s["sel"], workspace=s["ws"])
    S.still_hybrid_attn_bwd(s["p"], s["q"], s["k"], s["v"], s["g"], s["Wq"], s["bq"], s["Wk"], s["bk"], s["out"],
                            s["dout"], s["lse"], s["sel"], g["dq"], g["dk"], g["dv"], g["dg"], g["dWq"], g["dbq"],
                            g["dWk"], g["dbk"], s["bws"])
    return {"out": s["out"], "lse": s["lse"], **g}


def _run_transfer(s):
    g = s["grads"]
    S.still_hybrid_attn_fwd(s["p"], s["q"], s["k"], s["v"], s["g"], s["Wq"], s["bq"], s["Wk"], s["bk"], s["out"],
                            sel_idx=s["sel"], workspace=s["ws"])
    S.still_attention_map(s["p"], s["q"], s["k"], s["Wq"], s["bq"], s["Wk"], s["bk"], s["lse"], s["sel"], s["map"],
                          s["bws"])
    S.still_attention_map_bwd(s["p"], s["q"], s["k"], s["Wq"], s["bq"], s["Wk"], s["bk"], s["lse"], s["sel"], s["map"],
                              s["dmap"], g["dWq"], g["dbq"], g["dWk"], g["dbk"], s["bws"])
    return {"out": s["out"], "map": s["map"], **g}


# ------------------------------------------------------------------ what a pass cannot do without

def _visible(case, n):
    """(row, key) pairs of the softmax branch of one head over rows 0..n-1: retained keys of chunks <= c-2, the previous
    chunk, the own chunk up to the row."""
    C, lam, total = case["C"], case["lam"], 0
    for c in range((n + C - 1) // C):
        rows = min(C, n - c * C)
        ret = max(0, c - 1) * lam
        if case["budget"]:
            ret = min(ret, case["budget"])
        total += rows * (ret + (C if c >= 1 else 0)) + rows * (rows + 1) // 2
    return total


def _fwd_work(case):
    """A prefill call: q, k, v (and the gate) read once, the output written once; score logits, both feature maps, the
    state update, phi_q S, and the softmax branch."""
    B, N, Hq, Hkv, d = case["B"], case["N"], case["Hq"], case["Hkv"], case["d"]
    es = 2 if case["dtype"] == "bf16" else 4
    rows = B * N * (0.75 if case["ragged"] else 1.0)         # (expected length of a right-padded batch)
    nbytes = rows * d * es * (2 * Hq + 2 * Hkv + (Hq if case["gate"] != "none" else 0)) + 2 * Hq * d * d * es
    flops = Hq * (rows * (2 * d * min(case["W"], N) + 12 * d * d) + rows / N * 4 * d * _visible(case, N))
    return nbytes, flops


def _decode_work(case, t):
    B, Hq, Hkv, d, C = case["B"], case["Hq"], case["Hkv"], case["d"], case["C"]
    es = 2 if case["dtype"] == "bf16" else 4
    c = t // C
    ret = max(0, c - 1) * case["lam"]
    if case["budget"]:
        ret = min(ret, case["budget"])
    loc = t - max(0, c - 1) * C + 1
    slices = Hkv if case["shared"] else Hq
    nbytes = B * (slices * ret * 2 * d * es + Hkv * loc * 2 * d * es + Hq * 2 * d * (d + 1) * 4) + Hq * d * d * es
    flops = B * Hq * (4 * d * (ret + loc) + 2 * d * d + 4 * d * d + 2 * d * min(case["W"], t + 1))
    return nbytes, flops


def work(case):
    B, N, Hq, Hkv, d = case["B"], case["N"], case["Hq"], case["Hkv"], case["d"]
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "decode":
        nbytes, flops = _decode_work(case, N)
        return {"bytes": nbytes, "flops": flops}
    nbytes, flops = _fwd_work(case)
    if case["kind"] == "generate":
        for i in range(case["steps"]):
            b, f = _decode_work(case, int(0.75 * N) + i)
            nbytes, flops = nbytes + b, flops + f
    elif case["kind"] == "train":
        # q, k, v, out, dout (and the gate) read, dq, dk, dv (dg) written; five products per visible pair, and 36 d d_f per
        # token and head in the linear branch
        gates = 2 * Hq if case["gate"] != "none" else 0
        nbytes += B * N * d * es * (3 * Hq + 2 * Hkv + Hq + 2 * Hkv + gates) + 2 * Hq * d * d * (es + 4)
        flops += Hq * B * (10 * d * _visible(case, N) + 36 * d * d * N)
    elif case["kind"] == "transfer":
        # the map written, then map and gradient read (at and below the diagonal); logits and phi_q . phi_k per pair, and
        # both products with the gradient of the weights
        pairs = N * (N + 1) / 2
        nbytes += B * Hq * (N * N + 2 * pairs) * 4 + 2 * B * N * d * es * (Hq + Hkv) + 2 * Hq * d * d * 4
        flops += B * Hq * (pairs * (2 * d + 4 * d + 8 * d) + 12 * d * d * N)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured: the bf16 path against the same path in fp32 storage on the same bf16 inputs differs by up to 3.8e-3 (2-norm
    # over 2-norm; dWk, dq; a single element of dq by 0.24 of the larger of itself and the root mean square), since operands
    # of the products (softmax weights, features, state images) and results are rounded to 8 bits, and at most 1.5e-5 of the
    # index lists differ (near-ties of the scores).  The fp32 path against the float64 oracle: 1e-6 to 2.5e-6 (sums of
    # thousands of terms, hardware exponentials).  Four times each.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 6e-5}
    return {"rel": 1.5e-2, "max": 0.95, "differ": 6e-5}

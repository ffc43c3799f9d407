"""GPU parity of the backward pass (still_hybrid_attn_bwd through the C ABI) against the float64 backward oracle on
the same seeded, dtype-rounded inputs, with the index lists the HIP forward pass chose.

Bars: every gradient tensor within 1e-4 of its largest magnitude on fp32 (measured ~1e-6), within 1e-2 of it on
bf16 (measured 2-5e-3: the operands of the matrix core and the stored results carry 8 bits of mantissa, the sums are
fp32); the log normaliser that the forward pass leaves for the backward pass within 1e-5 relative (fp32) / 2e-2
absolute (bf16).  dk, dv are compared after the oracle's per-head parts are added up over the query heads of a kv
head, parameter gradients after adding up the batch."""
import numpy as np
import pytest

from oracle import still_backward as OB
from paper_2602_02180_amd import binding as S
from paper_2602_02180_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

BAR = {"f32": 1e-4, "bf16": 1e-2}


def small(name, **kw):
    base = dict(B=1, N=512, Hq=2, Hkv=1, d=64, C=64, W=64, lam=16, dtype="f32")
    base.update(kw)
    return synth.Workload(name, **base)


def make_dy(w, inp, seed):
    rng = np.random.default_rng(seed)
    return synth.round_to_dtype(rng.standard_normal(inp["q"].shape).astype(np.float32), w.dtype)


def oracle_grads(w, inp, dy, sel, kv_map, gate_activation="none"):
    B, N = inp["q"].shape[:2]
    units = [(b, h) for b in range(B) for h in range(w.Hq)]
    ref = OB.still_backward_units(inp, dy.astype(np.float64), kv_map, units, w.C, w.W, w.lam, w.scale, w.eps,
                                  sel, max_retained=U.budget(w), gate_activation=gate_activation)
    g = {"dq": np.zeros(inp["q"].shape), "dk": np.zeros(inp["k"].shape), "dv": np.zeros(inp["v"].shape),
         "dWq": np.zeros(inp["Wq"].shape), "dWk": np.zeros(inp["Wk"].shape),
         "lse": np.zeros((B, w.Hq, N)),
         "dg": np.zeros(inp["q"].shape) if inp.get("g") is not None else None,
         "dbq": np.zeros((w.Hq, w.df)) if inp.get("bq") is not None else None,
         "dbk": np.zeros((w.Hq, w.df)) if inp.get("bk") is not None else None}
    for (b, h) in units:
        r = ref[(b, h)]
        kh = int(kv_map[h])
        g["dq"][b, :, h] = r["dq"]
        g["dk"][b, :, kh] += r["dk"]
        g["dv"][b, :, kh] += r["dv"]
        g["dWq"][h] += r["dWq"]
        g["dWk"][h] += r["dWk"]
        g["lse"][b, h] = r["lse"]
        for name in ("dg",):
            if g[name] is not None:
                g[name][b, :, h] = r[name]
        for name in ("dbq", "dbk"):
            if g[name] is not None:
                g[name][h] += r[name]
    return g


def check_backward(w, inp, seed, kv_map=None, gate_activation=0):
    kv = synth.kv_head_map(w) if kv_map is None else kv_map
    dy = make_dy(w, inp, seed)
    hip = U.run_hip_backward(w, inp, dy, kv_map=kv_map, gate_activation=gate_activation)
    ref = oracle_grads(w, inp, dy, hip["sel"], kv, "sigmoid" if gate_activation else "none")
    lse_err = float(np.max(np.abs(hip["lse"] - ref["lse"])))
    print(f"[{w.name}] lse max-abs err {lse_err:.3e}")
    assert lse_err <= (1e-5 * max(1.0, float(np.max(np.abs(ref["lse"])))) if w.dtype == "f32" else 2e-2)
    worst = {}
    for name in ("dq", "dk", "dv", "dg", "dWq", "dWk", "dbq", "dbk"):
        if ref[name] is None:
            assert hip[name] is None
            continue
        x = hip[name].astype(np.float64)
        assert np.all(np.isfinite(x)), name
        scale = float(np.max(np.abs(ref[name])))
        err = float(np.max(np.abs(x - ref[name])))
        worst[name] = err / max(scale, 1e-30) if scale > 0 else err
        print(f"[{w.name}] {name}: max |ref| {scale:.3e}  max-abs err {err:.3e}  ratio {worst[name]:.3e}")
    for name, r in worst.items():
        assert r <= BAR[w.dtype], (name, r)
    return hip, ref


def with_bias(w, inp, seed):
    rng = np.random.default_rng(seed)
    inp["bq"] = synth.round_to_dtype(rng.standard_normal((w.Hq, w.df)) * 0.1, w.dtype)
    inp["bk"] = synth.round_to_dtype(rng.standard_normal((w.Hq, w.df)) * 0.1, w.dtype)
    return inp


def test_backward_fp32_gate_bias_gqa_ragged_tail():
    w = small("bwd", N=600, Hq=4, Hkv=2, lam=8, B=2)
    inp = with_bias(w, synth.make_inputs(w, seed=31, with_gate=True), 32)
    hip, ref = check_backward(w, inp, 33)
    # both branches are live: no gradient is identically zero
    for name in ("dq", "dk", "dv", "dg", "dWq", "dWk", "dbq", "dbk"):
        assert np.max(np.abs(ref[name])) > 1e-4, name


@pytest.mark.parametrize("kw", [
    dict(N=512, lam=16, max_retained=40),                 # the budget runs out in chunk 2
    dict(N=384, lam=0),                                   # nothing retained: local span + linear state only
    dict(N=320, lam=64),                                  # everything retained: no linear branch at all
    dict(N=50),                                           # shorter than one chunk
    dict(N=1024, C=128, W=128, lam=16, Hq=2, Hkv=2),      # the wide chunk
    dict(N=2304, lam=4, Hq=1),                            # many chunks: several segments of the state scan
], ids=["budget", "lam0", "all-kept", "short", "C128", "segments"])
def test_backward_fp32_cases(kw):
    w = small("bwd-" + "-".join(f"{k}{v}" for k, v in kw.items()), **kw)
    check_backward(w, synth.make_inputs(w, seed=41, with_gate=True), 42)


def test_backward_fp32_sigmoid_gate_and_custom_head_map():
    w = small("bwd-sg", N=448, Hq=4, Hkv=2, lam=8)
    inp = synth.make_inputs(w, seed=51)
    rng = np.random.default_rng(52)
    inp["g"] = synth.round_to_dtype(2.0 * rng.standard_normal(inp["q"].shape), w.dtype)
    check_backward(w, inp, 53, kv_map=np.array([1, 0, 0, 1], np.int32), gate_activation=1)


@pytest.mark.parametrize("kw", [
    dict(d=128, C=128, W=128, N=1024, Hq=4, Hkv=2),
    dict(d=64, C=64, W=64, N=1100, Hq=4, Hkv=1, B=2),
    dict(d=128, C=64, W=128, N=900, Hq=2, Hkv=1, max_retained=96),
    dict(d=64, C=128, W=256, N=1500, Hq=3, Hkv=1, B=3, lam=32, max_retained=70),
], ids=["d128-C128", "d64-ragged", "d128-budget", "d64-C128-budget-wide-window"])
def test_backward_bf16(kw):
    w = small("bwd16-" + "-".join(f"{k}{v}" for k, v in kw.items()), dtype="bf16", **kw)
    inp = with_bias(w, synth.make_inputs(w, seed=61, with_gate=True), 62)
    check_backward(w, inp, 63)


@pytest.mark.parametrize("kw", [
    dict(dtype="bf16", d=128, N=31, lam=4),                          # one ragged 32-row tile
    dict(dtype="bf16", d=128, N=129, lam=4, Hq=4),                   # one row past a 128-row / 128-key workgroup
    dict(dtype="bf16", d=64, N=64 * 21 + 33, lam=7),                 # 133 visible entries: just past a 128-entry tile
    dict(dtype="f32", N=64 * 10, lam=16, Hq=3),                      # exactly 128 visible entries
    dict(dtype="bf16", d=128, C=128, N=128 * 5 - 1, lam=128),        # every token retained, last chunk ragged
], ids=["n31", "n129", "entries133", "entries128", "all-kept-ragged"])
def test_backward_at_the_edges_of_the_softmax_tiles(kw):
    w = small("bwd-edge-" + "-".join(f"{k}{v}" for k, v in kw.items()), **kw)
    check_backward(w, synth.make_inputs(w, seed=71, with_gate=True), 72)


def test_backward_at_the_training_shape_sampled_units():
    """Config c6 (the shape bench.py --backward times: 16 sequences of 1024 tokens, 32 query heads over 8 kv heads,
    d = 128, bf16), in the launch configuration the benchmark uses.  The oracle covers what it can reach in seconds:
    dq and dg of the four query heads of kv head 2 in sequence 5, dk and dv of that kv head (the sum over exactly
    those four heads), and dWq, dWk, of query head 9 (sums over all 16 sequences)."""
    w = synth.workload("c6")
    inp = synth.make_inputs(w, with_gate=True)
    dy = make_dy(w, inp, 71)
    hip = U.run_hip_backward(w, inp, dy)
    kv = synth.kv_head_map(w)
    b, kh = 5, 2
    heads = [h for h in range(w.Hq) if kv[h] == kh]
    units = [(b, h) for h in heads] + [(bb, 9) for bb in range(w.B)]
    ref = OB.still_backward_units(inp, dy.astype(np.float64), kv, units, w.C, w.W, w.lam, w.scale, w.eps, hip["sel"])
    bar = BAR[w.dtype]

    def check(name, x, y):
        scale = float(np.max(np.abs(y)))
        err = float(np.max(np.abs(x.astype(np.float64) - y)))
        print(f"[c6] {name}: max |ref| {scale:.3e}  max-abs err {err:.3e}  ratio {err / scale:.3e}")
        assert np.all(np.isfinite(x)) and err <= bar * scale, (name, err, scale)

    for h in heads:
        check(f"dq head {h}", hip["dq"][b, :, h], ref[(b, h)]["dq"])
        check(f"dg head {h}", hip["dg"][b, :, h], ref[(b, h)]["dg"])
    check("dk", hip["dk"][b, :, kh], sum(ref[(b, h)]["dk"] for h in heads))
    check("dv", hip["dv"][b, :, kh], sum(ref[(b, h)]["dv"] for h in heads))
    check("dWq head 9", hip["dWq"][9], sum(ref[(bb, 9)]["dWq"] for bb in range(w.B)))
    check("dWk head 9", hip["dWk"][9], sum(ref[(bb, 9)]["dWk"] for bb in range(w.B)))


def test_backward_with_group_shared_selection_bf16():
    """The selection variant only changes WHICH tokens are kept (one list per kv head); the backward pass takes the
    lists as they are."""
    w = small("bwd-shared", dtype="bf16", d=64, N=768, Hq=4, Hkv=2, lam=8, shared_selection=True)
    inp = synth.make_inputs(w, seed=81, with_gate=True)
    hip, _ = check_backward(w, inp, 82)
    assert np.array_equal(hip["sel"][:, 0], hip["sel"][:, 1]) and np.array_equal(hip["sel"][:, 2], hip["sel"][:, 3])


def test_backward_twice_on_a_user_stream_gives_the_same_gradients():
    """Nothing in the workspace has to start at zero and nothing survives a call: a second call into the same
    (dirty) workspace on a non-default stream reproduces the first to rounding (the parameter gradients are summed
    with atomic adds, so not bit for bit)."""
    import torch

    w = small("bwd-twice", N=700, Hq=4, Hkv=2, lam=8)
    inp = synth.make_inputs(w, seed=91, with_gate=True)
    dy = make_dy(w, inp, 92)
    dev = "cuda"
    q, k, v, g, Wq, Wk = (synth.to_torch(inp[n], w.dtype, dev) for n in ("q", "k", "v", "g", "Wq", "Wk"))
    dout = synth.to_torch(dy, w.dtype, dev)
    out = torch.empty_like(q)
    p = S.make_params(B=w.B, N=w.N, Hq=w.Hq, Hkv=w.Hkv, d=w.d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps,
                      dtype=w.dtype, q=q, k=k, v=v, out=out, g=g)
    sel = torch.zeros(w.B, w.Hq, w.N // w.C, w.lam, dtype=torch.int32, device=dev)
    ws = torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device=dev)
    bws = torch.empty(S.still_bwd_workspace_bytes(p), dtype=torch.uint8, device=dev)
    L = S.still_fwd_workspace_layout(p)
    lse = ws[L.lse:L.lse + w.B * w.Hq * w.N * 4].view(torch.float32)
    stream = torch.cuda.Stream()
    results = []
    with torch.cuda.stream(stream):
        S.still_hybrid_attn_fwd(p, q, k, v, g, Wq, None, Wk, None, out, sel_idx=sel, workspace=ws, stream=stream)
        for _ in range(2):
            grads = [torch.full_like(t, float("nan")) for t in (q, k, v, g)]
            dWq = torch.full((w.Hq, w.d, w.d), float("nan"), dtype=torch.float32, device=dev)
            dWk = torch.full_like(dWq, float("nan"))
            S.still_hybrid_attn_bwd(p, q, k, v, g, Wq, None, Wk, None, out, dout, lse, sel, grads[0], grads[1], grads[2],
                                    grads[3], dWq, None, dWk, None, bws, stream=stream)
            results.append([t.clone() for t in grads + [dWq, dWk]])
    stream.synchronize()
    for a_, b_ in zip(*results):
        a_, b_ = a_.float(), b_.float()
        assert torch.isfinite(a_).all() and torch.isfinite(b_).all()
        assert float((a_ - b_).abs().max()) <= 1e-5 * float(a_.abs().max())


@pytest.mark.parametrize("kw", [
    dict(dtype="f32", N=600, Hq=4, Hkv=2, lam=8, B=2),
    dict(dtype="f32", N=512, lam=16, max_retained=40),
    dict(dtype="bf16", d=128, C=128, W=128, N=1024, Hq=4, Hkv=2),
    dict(dtype="f32", N=50),                               # shorter than a chunk: no linear branch, 56-column rows
    dict(dtype="bf16", d=64, N=330, lam=4, Hq=3, Hkv=3, B=3),
], ids=["f32-gqa-ragged", "f32-budget", "bf16-d128", "f32-short", "bf16-odd-sizes"])
def test_attention_map_against_the_oracle(kw):
    """still_attention_map for the forward call's lists and normalisers: element-wise against the oracle's map
    (weights are at most one: absolute bars 2e-6 on fp32, 4e-3 on bf16, whose logits and features carry 8 bits),
    rows sum to one, nothing above the diagonal, and map x v reproduces the forward output (no gate)."""
    import torch

    w = small("map-" + "-".join(f"{k}{v}" for k, v in kw.items()), **kw)
    inp = with_bias(w, synth.make_inputs(w, seed=101), 102)
    dev = "cuda"
    up = lambda n: synth.to_torch(inp[n], w.dtype, dev)
    q, k, v, Wq, Wk, bq, bk = (up(n) for n in ("q", "k", "v", "Wq", "Wk", "bq", "bk"))
    B, N = q.shape[:2]
    out = torch.empty_like(q)
    p = S.make_params(B=B, N=N, Hq=w.Hq, Hkv=w.Hkv, d=w.d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps,
                      dtype=w.dtype, q=q, k=k, v=v, out=out, max_retained=w.max_retained)
    sel = torch.full((B, w.Hq, N // w.C, w.lam), -1, dtype=torch.int32, device=dev)
    ws = torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device=dev)
    S.still_hybrid_attn_fwd(p, q, k, v, None, Wq, bq, Wk, bk, out, sel_idx=sel, workspace=ws)
    L = S.still_fwd_workspace_layout(p)
    lse = ws[L.lse:L.lse + B * w.Hq * N * 4].view(torch.float32)
    amap = torch.full((B, w.Hq, N, N), float("nan"), dtype=torch.float32, device=dev)
    bws = torch.empty(S.still_bwd_workspace_bytes(p), dtype=torch.uint8, device=dev)
    S.still_attention_map(p, q, k, Wq, bq, Wk, bk, lse, sel, amap, bws)
    torch.cuda.synchronize()
    A = amap.cpu().numpy().astype(np.float64)
    sel_h = sel.cpu().numpy().astype(np.int64)
    y = synth.from_torch(out).astype(np.float64)
    kv = synth.kv_head_map(w)
    bar = 2e-6 if w.dtype == "f32" else 4e-3
    assert np.all(np.isfinite(A)) and np.all(np.triu(A, 1) == 0.0)
    worst = 0.0
    for b in range(B):
        for h in range(w.Hq):
            ref = OB.attention_map(inp["q"][b, :, h], inp["k"][b, :, kv[h]], inp["Wq"][h], inp["Wk"][h], w.C, w.W, w.lam,
                                   w.scale, w.eps, bq=inp["bq"][h], bk=inp["bk"][h], sel=sel_h[b, h],
                                   max_retained=U.budget(w))
            worst = max(worst, float(np.max(np.abs(A[b, h] - ref))))
            assert np.max(np.abs(A[b, h].sum(axis=1) - 1.0)) <= (1e-5 if w.dtype == "f32" else 1e-2)
            yv = A[b, h] @ inp["v"][b, :, kv[h]].astype(np.float64)
            if w.dtype == "f32":
                assert U.rel_err(yv, y[b, :, h]) <= 1e-4
    print(f"[{w.name}] attention map: max-abs err {worst:.3e}")
    assert worst <= bar, worst
    # and its backward pass to the feature-map parameters, for a random dmap
    rng = np.random.default_rng(103)
    dA = np.tril(rng.standard_normal((B, w.Hq, N, N)).astype(np.float32))
    dmap = torch.from_numpy(dA).to(dev)
    f32 = dict(dtype=torch.float32, device=dev)
    dWq, dWk = torch.full((w.Hq, w.d, w.df), float("nan"), **f32), torch.full((w.Hq, w.d, w.df), float("nan"), **f32)
    dbq, dbk = torch.full((w.Hq, w.df), float("nan"), **f32), torch.full((w.Hq, w.df), float("nan"), **f32)
    mws = torch.empty(S.still_attention_map_bwd_workspace_bytes(p), dtype=torch.uint8, device=dev)
    S.still_attention_map_bwd(p, q, k, Wq, bq, Wk, bk, lse, sel, amap, dmap, dWq, dbq, dWk, dbk, mws)
    torch.cuda.synchronize()
    ref = {n: np.zeros(s_) for n, s_ in (("dWq", (w.Hq, w.d, w.df)), ("dWk", (w.Hq, w.d, w.df)), ("dbq", (w.Hq, w.df)),
                                         ("dbk", (w.Hq, w.df)))}
    for b in range(B):
        for h in range(w.Hq):
            r = OB.attention_map_backward(inp["q"][b, :, h], inp["k"][b, :, kv[h]], inp["Wq"][h], inp["Wk"][h], w.C, w.W,
                                          w.lam, w.scale, w.eps, dA[b, h].astype(np.float64), bq=inp["bq"][h],
                                          bk=inp["bk"][h], sel=sel_h[b, h], max_retained=U.budget(w))
            for n in ref:
                ref[n][h] += r[n]
    for n, t in (("dWq", dWq), ("dWk", dWk), ("dbq", dbq), ("dbk", dbk)):
        x = t.cpu().numpy().astype(np.float64)
        scale_ = float(np.max(np.abs(ref[n])))
        err = float(np.max(np.abs(x - ref[n])))
        print(f"[{w.name}] map backward {n}: max |ref| {scale_:.3e}  max-abs err {err:.3e}")
        assert np.all(np.isfinite(x)) and err <= BAR[w.dtype] * max(scale_, 1e-30), (n, err, scale_)


@pytest.mark.parametrize("kw,gate", [
    (dict(dtype="bf16", d=128, C=128, N=128 * 9 + 70, Hq=8, Hkv=2, lam=8), True),   # two 64-token tiles per image, prefix images
    (dict(dtype="bf16", d=128, C=64, N=64 * 3, Hq=8, Hkv=8, lam=5), False),         # one chunk with a state behind it, no gate
    (dict(dtype="bf16", d=64, C=64, N=64 * 7 + 1, Hq=6, Hkv=2, lam=16), True),      # a last tile of one token
    (dict(dtype="f32", C=64, N=64 * 5 + 63, Hq=8, Hkv=4, lam=3), False),            # a last tile short of one token
    (dict(dtype="f32", C=128, W=128, N=128 * 6 - 64, Hq=2, Hkv=2, lam=16), True),   # the last chunk is half a chunk
], ids=["bf16-d128-C128", "bf16-no-gate-3-chunks", "bf16-d64-one-token-tail", "f32-no-gate", "f32-C128-half-chunk"])
def test_backward_linear_branch_tiles(kw, gate):
    """The linear branch works in tiles of 64 tokens (several kv groups and their head maps, both image sources)."""
    w = small("bwd-lin-" + "-".join(f"{k}{v}" for k, v in kw.items()), **kw)
    check_backward(w, with_bias(w, synth.make_inputs(w, seed=81, with_gate=gate), 82), 83)


@pytest.mark.parametrize("kw", [
    dict(dtype="f32", C=64, N=64 * 5 + 1, Hq=4, Hkv=2, lam=8),                   # rows that start on any 4-byte boundary, a tile of one row
    dict(dtype="f32", C=128, W=128, N=128 * 4 + 62, Hq=8, Hkv=8, lam=16),        # two tiles per chunk, eight units (XCD order)
    dict(dtype="bf16", d=128, C=64, N=64 * 3, Hq=2, Hkv=1, lam=4, B=4),          # one chunk of pairs: a single tile either side
    dict(dtype="bf16", d=128, C=128, W=128, N=128 * 5 - 3, Hq=3, Hkv=3, lam=0),  # nothing selected, a last chunk short of three
], ids=["f32-one-row-tail", "f32-C128", "bf16-one-tile", "bf16-none-selected"])
def test_attention_map_tiles(kw):
    """The map and its backward pass work in tiles of 64 rows and 64 keys."""
    test_attention_map_against_the_oracle(kw)


@pytest.mark.parametrize("over", [
    dict(dq="q", dk="k", dv="v"), dict(dk="v", dv="k"), dict(dq="k"), dict(dq="dout", dg="g"), dict(dg="dout"), dict(dk="out", dv="q"),
], ids=lambda o: "-".join(f"{a}_over_{b}" for a, b in o.items()))
@pytest.mark.parametrize("kw", [dict(dtype="f32", N=64 * 9 + 5), dict(dtype="bf16", d=128, C=128, W=128, N=128 * 6 + 40)],
                         ids=["f32", "bf16-C128"])
def test_backward_results_may_lie_over_its_inputs(kw, over):
    """The call reads every input before it writes over one, so gradients may share memory with inputs.  dq, dk, dv and dg
    are sums in a fixed order, rounded once: bit for bit those of a call with separate tensors; the parameter gradients
    are added atomically (1e-5 of the largest)."""
    import torch

    w = small("bwd-over", **dict(dict(Hq=4, Hkv=4, lam=8, B=2), **kw))
    inp = synth.make_inputs(w, seed=121, with_gate=True)
    t = {n: synth.to_torch(inp[n], w.dtype, "cuda") for n in ("q", "k", "v", "g", "Wq", "Wk")}
    t["dout"], t["out"] = synth.to_torch(make_dy(w, inp, 122), w.dtype, "cuda"), torch.empty_like(t["q"])
    p = S.make_params(B=w.B, N=w.N, Hq=w.Hq, Hkv=w.Hkv, d=w.d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps,
                      dtype=w.dtype, q=t["q"], k=t["k"], v=t["v"], out=t["out"], g=t["g"])
    sel = torch.zeros(w.B, w.Hq, w.N // w.C, w.lam, dtype=torch.int32, device="cuda")
    ws = torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.still_hybrid_attn_fwd(p, t["q"], t["k"], t["v"], t["g"], t["Wq"], None, t["Wk"], None, t["out"], sel_idx=sel, workspace=ws)
    off = S.still_fwd_workspace_layout(p).lse
    lse = ws[off:off + w.B * w.Hq * w.N * 4].view(torch.float32)

    def backward(over):
        x = {n: y.clone() for n, y in t.items()}
        res = {a: x[over[a]] if a in over else torch.full_like(t[b], float("nan"))
               for a, b in (("dq", "q"), ("dk", "k"), ("dv", "v"), ("dg", "g"))}
        res.update({n: torch.full((w.Hq, w.d, w.d), float("nan"), dtype=torch.float32, device="cuda") for n in ("dWq", "dWk")})
        bws = torch.full((S.still_bwd_workspace_bytes(p),), 0x7f, dtype=torch.uint8, device="cuda")
        S.still_hybrid_attn_bwd(p, x["q"], x["k"], x["v"], x["g"], x["Wq"], None, x["Wk"], None, x["out"], x["dout"], lse, sel,
                                res["dq"], res["dk"], res["dv"], res["dg"], res["dWq"], None, res["dWk"], None, bws)
        torch.cuda.synchronize()
        return res

    want, got = backward({}), backward(over)
    for n in ("dq", "dk", "dv", "dg"):
        differ = int((got[n] != want[n]).sum())
        assert differ == 0, n
    for n in ("dWq", "dWk"):
        err = float((got[n] - want[n]).abs().max()) / float(want[n].abs().max())
        assert err <= 1e-5, n


@pytest.mark.parametrize("slots", [[5, 5, 9, 20, 20, 63], [63, 5, 9, 5, 20, 20], [40, 2, 31, 33, 0, 7]],
                         ids=["repeated", "repeated-unordered", "unordered"])
def test_backward_counts_every_entry_of_a_list(slots):
    """Lists that name a token twice, or not in ascending order: the softmax branch sees every entry, so every entry has a
    gradient.  Against torch's autograd on the output equation in float64 with the entries written out."""
    import torch

    w = small("bwd-entries", N=64 * 5 + 10, Hq=2, Hkv=1, lam=len(slots))
    inp = synth.make_inputs(w, seed=131)
    t = {n: synth.to_torch(inp[n], w.dtype, "cuda") for n in ("q", "k", "v", "Wq", "Wk")}
    dy = make_dy(w, inp, 132)
    dout, out = synth.to_torch(dy, w.dtype, "cuda"), torch.empty_like(t["q"])
    p = S.make_params(B=1, N=w.N, Hq=w.Hq, Hkv=w.Hkv, d=w.d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps,
                      dtype=w.dtype, q=t["q"], k=t["k"], v=t["v"], out=out)
    lists = torch.tensor([[c * w.C + x for x in slots] for c in range(w.N // w.C)], dtype=torch.int32)
    sel = lists.expand(1, w.Hq, *lists.shape).contiguous().cuda()
    ws = torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.still_hybrid_attn_fwd(p, t["q"], t["k"], t["v"], None, t["Wq"], None, t["Wk"], None, out, sel_idx=sel, workspace=ws,
                            sel_idx_is_input=1)
    off = S.still_fwd_workspace_layout(p).lse
    lse = ws[off:off + w.Hq * w.N * 4].view(torch.float32)
    got = {"d" + n: torch.full_like(t[n], float("nan"), dtype=torch.float32) for n in t}
    bws = torch.empty(S.still_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.still_hybrid_attn_bwd(p, t["q"], t["k"], t["v"], None, t["Wq"], None, t["Wk"], None, out, dout, lse, sel, got["dq"],
                            got["dk"], got["dv"], None, got["dWq"], None, got["dWk"], None, bws)

    x = {n: y.detach().cpu().double().requires_grad_() for n, y in t.items()}

    def features(a, W):
        f = a @ W
        u = f / f.norm(dim=-1, keepdim=True) * a.norm(dim=-1, keepdim=True)
        return torch.cat([u.softmax(-1), (-u).softmax(-1)], -1)

    # how often every row sees every key through exp; what it does not see of the routed chunks goes through phi
    tok = torch.arange(w.N)
    c, j = tok[:, None] // w.C, tok[None, :]
    count = torch.bincount(lists.flatten().long(), minlength=w.N).double()
    routed = j // w.C <= c - 2
    seen = torch.where(routed, count[None, :], ((j // w.C >= c - 1) & (j <= tok[:, None])).double())
    k, v = x["k"][0, :, 0], x["v"][0, :, 0]
    y = []
    for h in range(w.Hq):
        q = x["q"][0, :, h]
        a = seen * torch.exp(w.scale * (q @ k.T)) + (routed & (count == 0)) * (features(q, x["Wq"][h]) @ features(k, x["Wk"][h]).T)
        y.append(a @ v / a.sum(-1, keepdim=True))
    torch.stack(y, 1)[None].backward(torch.from_numpy(dy).double())
    for n in t:
        ref = x[n].grad
        err = float((got["d" + n].cpu().double() - ref).abs().max()) / float(ref.abs().max())
        assert err <= BAR["f32"], ("d" + n, err)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_backward_makes_no_transposed_copy_of_v(dtype, d):
    """The state scan reads v in operand order only: region `vt` of the workspace keeps what it held."""
    import torch

    w = small("bwd-vt", dtype=dtype, d=d, N=450, Hq=2, Hkv=2, lam=4)
    inp = synth.make_inputs(w, seed=141)
    q, k, v, Wq, Wk = (synth.to_torch(inp[n], w.dtype, "cuda") for n in ("q", "k", "v", "Wq", "Wk"))
    out, lse = torch.zeros_like(q), torch.zeros(w.Hq * w.N, dtype=torch.float32, device="cuda")
    p = S.make_params(B=1, N=w.N, Hq=w.Hq, Hkv=w.Hkv, d=d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps, dtype=dtype,
                      q=q, k=k, v=v, out=out)
    sel = torch.arange(w.N // w.C, device="cuda", dtype=torch.int32)[:, None] * w.C + torch.arange(w.lam, device="cuda", dtype=torch.int32)
    sel = sel.expand(1, w.Hq, *sel.shape).contiguous()
    bws = torch.full((S.still_bwd_workspace_bytes(p),), 0x5a, dtype=torch.uint8, device="cuda")
    dq, dk, dv = (torch.empty_like(x) for x in (q, k, v))
    dWq, dWk = (torch.empty(w.Hq, d, d, dtype=torch.float32, device="cuda") for _ in range(2))
    S.still_hybrid_attn_bwd(p, q, k, v, None, Wq, None, Wk, None, out, out, lse, sel, dq, dk, dv, None, dWq, None, dWk, None, bws)
    L = S.still_fwd_workspace_layout(p)
    untouched = bool((bws[L.vt:L.kret] == 0x5a).all())
    assert untouched


@pytest.mark.parametrize("kw", [
    dict(dtype="f32", N=64 * 6 + 9, Hq=4, Hkv=2), dict(dtype="bf16", d=128, C=128, W=128, N=128 * 5 - 30, Hq=2, Hkv=2),
    dict(dtype="bf16", N=64 * 5, Hq=8, Hkv=1)], ids=["f32", "bf16-C128", "bf16-d64"])
def test_backward_and_map_with_strided_tensors(kw):
    """q, k and v as slices of one packed projection, out and dout head-major, the gate with gaps between its rows: bit for bit
    the gradients and the map of contiguous tensors (every sum runs in the same order; the parameter gradients are
    added atomically: 1e-5 of the largest), and nothing between the rows is written."""
    import torch

    w = small("bwd-strided", **dict(dict(lam=8, B=2), **kw))
    B, N, Hq, Hkv, d = w.B, w.N, w.Hq, w.Hkv, w.d
    inp = synth.make_inputs(w, seed=151, with_gate=True)
    t = {n: synth.to_torch(inp[n], w.dtype, "cuda") for n in ("q", "k", "v", "g", "Wq", "Wk")}
    t["dout"] = synth.to_torch(make_dy(w, inp, 152), w.dtype, "cuda")
    dt = t["q"].dtype

    def packed(fill):                                    # [B, N, (Hq + 2 Hkv + 1) d]: q, k, v and a column block of nothing
        x = torch.full((B, N, Hq + 2 * Hkv + 1, d), fill, dtype=dt, device="cuda")
        return x, x[:, :, :Hq], x[:, :, Hq:Hq + Hkv], x[:, :, Hq + Hkv:Hq + 2 * Hkv]

    def run(strided):
        junk = []
        if strided:
            _, q, k, v = packed(7.0)
            grads, dq, dk, dv = packed(5.0)
            out, dout = (torch.empty(B, Hq, N, d, dtype=dt, device="cuda").permute(0, 2, 1, 3) for _ in range(2))
            g, dg = (torch.full((B, N, Hq, d + 16), x, dtype=dt, device="cuda") for x in (7.0, 5.0))
            junk = [grads[:, :, Hq + 2 * Hkv:], dg[..., d:]]
            g, dg = g[..., :d], dg[..., :d]
        else:
            q, k, v, g, dout, out = (torch.empty_like(t[n]) for n in ("q", "k", "v", "g", "dout", "dout"))
            dq, dk, dv, dg = (torch.empty_like(x) for x in (q, k, v, g))
        for n, x in (("q", q), ("k", k), ("v", v), ("g", g), ("dout", dout)):
            x.copy_(t[n])
        p = S.make_params(B=B, N=N, Hq=Hq, Hkv=Hkv, d=d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps, dtype=w.dtype, q=q,
                          k=k, v=v, out=out, g=g)
        sel = torch.zeros(B, Hq, N // w.C, w.lam, dtype=torch.int32, device="cuda")
        ws = torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        S.still_hybrid_attn_fwd(p, q, k, v, g, t["Wq"], None, t["Wk"], None, out, sel_idx=sel, workspace=ws)
        off = S.still_fwd_workspace_layout(p).lse
        lse = ws[off:off + B * Hq * N * 4].view(torch.float32)
        dWq, dWk, mWq, mWk = (torch.empty(Hq, d, d, dtype=torch.float32, device="cuda") for _ in range(4))
        bws = torch.empty(S.still_attention_map_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        S.still_hybrid_attn_bwd(p, q, k, v, g, t["Wq"], None, t["Wk"], None, out, dout, lse, sel, dq, dk, dv, dg, dWq, None, dWk,
                                None, bws)
        amap = torch.empty(B, Hq, N, N, dtype=torch.float32, device="cuda")
        S.still_attention_map(p, q, k, t["Wq"], None, t["Wk"], None, lse, sel, amap, bws)
        S.still_attention_map_bwd(p, q, k, t["Wq"], None, t["Wk"], None, lse, sel, amap, amap.square(), mWq, None, mWk, None, bws)
        return dict(out=out, dq=dq, dk=dk, dv=dv, dg=dg, map=amap), dict(dWq=dWq, dWk=dWk, mWq=mWq, mWk=mWk), junk

    (same, near, _), (same_s, near_s, junk) = run(False), run(True)
    for n in same:
        differ = int((same[n] != same_s[n]).sum())
        assert differ == 0, n
    for n in near:
        err = float((near[n] - near_s[n]).abs().max()) / float(near[n].abs().max())
        assert err <= 1e-5, (n, err)
    for x in junk:
        kept = bool((x == 5.0).all())
        assert kept


@pytest.mark.parametrize("kw", [dict(dtype="f32", N=64 * 4 + 3), dict(dtype="bf16", d=128, C=64, N=64 * 8 + 61),
                                dict(dtype="bf16", d=64, C=128, W=128, N=128 * 5)], ids=["f32-259", "bf16-573", "bf16-640"])
def test_map_backward_reads_nothing_above_the_diagonal(kw):
    """The row sums take whole pieces of a row and drop the columns behind the diagonal, the last piece lies inside the
    row: NaN above the diagonal of both matrices changes no gradient (added atomically: 1e-5 of the largest)."""
    import torch

    w = small("map-nan", **dict(dict(Hq=3, Hkv=1, lam=8, B=2), **kw))
    inp = synth.make_inputs(w, seed=171)
    t = {n: synth.to_torch(inp[n], w.dtype, "cuda") for n in ("q", "k", "v", "Wq", "Wk")}
    out = torch.empty_like(t["q"])
    p = S.make_params(B=w.B, N=w.N, Hq=w.Hq, Hkv=w.Hkv, d=w.d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps,
                      dtype=w.dtype, q=t["q"], k=t["k"], v=t["v"], out=out)
    sel = torch.zeros(w.B, w.Hq, w.N // w.C, w.lam, dtype=torch.int32, device="cuda")
    ws = torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.still_hybrid_attn_fwd(p, t["q"], t["k"], t["v"], None, t["Wq"], None, t["Wk"], None, out, sel_idx=sel, workspace=ws)
    L = S.still_fwd_workspace_layout(p)
    lse = ws[L.lse:L.lse + w.B * w.Hq * w.N * 4].view(torch.float32)
    amap = torch.empty(w.B, w.Hq, w.N, w.N, device="cuda")
    bws = torch.empty(S.still_attention_map_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.still_attention_map(p, t["q"], t["k"], t["Wq"], None, t["Wk"], None, lse, sel, amap, bws)
    g = torch.Generator(device="cuda")
    g.manual_seed(172)
    dmap = torch.randn(amap.shape, generator=g, device="cuda").tril_()
    upper = torch.ones(w.N, w.N, dtype=torch.bool, device="cuda").triu_(1)
    grads = []
    for fill in (0.0, float("nan")):
        dWq, dWk = torch.empty(w.Hq, w.d, w.d, device="cuda"), torch.empty(w.Hq, w.d, w.d, device="cuda")
        S.still_attention_map_bwd(p, t["q"], t["k"], t["Wq"], None, t["Wk"], None, lse, sel, amap.masked_fill(upper, fill),
                                  dmap.masked_fill(upper, fill), dWq, None, dWk, None, bws)
        grads.append((dWq, dWk))
    for a_, b_ in zip(*grads):
        assert torch.isfinite(b_).all() and float(a_.abs().max()) > 0
        assert float((a_ - b_).abs().max()) <= 1e-5 * float(a_.abs().max())


@pytest.mark.parametrize("kw,kv_map", [
    (dict(dtype="bf16", d=64, N=64 * 6 + 9, Hq=11, Hkv=2, lam=16), [0, 1, 0, 0, 1, 0, 0, 0, 0, 0, 0]),   # groups of nine and two, interleaved
    (dict(dtype="f32", N=64 * 5, Hq=6, Hkv=1, lam=64), None),                                            # every token retained, six heads
    (dict(dtype="bf16", d=128, C=128, W=128, N=128 * 5 + 70, Hq=5, Hkv=1, lam=128, max_retained=200), None),
    (dict(dtype="bf16", d=64, N=64 * 24 + 5, Hq=6, Hkv=1, lam=32, max_retained=64), None),               # most chunks keep nothing
], ids=["bf16-groups-of-9-and-2", "f32-all-kept", "bf16-C128-budget-inside-a-chunk", "bf16-budget-of-two-chunks"])
def test_backward_retained_entries_of_wide_groups(kw, kv_map):
    """The key side adds the retained entries of four query heads at a time, from a table of one slot per token and head."""
    w = small("bwd-ret-" + "-".join(f"{k}{v}" for k, v in kw.items()), **kw)
    inp = synth.make_inputs(w, seed=181, with_gate=True)
    check_backward(w, inp, 182, kv_map=None if kv_map is None else np.array(kv_map, np.int32))


@pytest.mark.parametrize("kw", [dict(dtype="f32", N=64 * 9 + 5), dict(dtype="bf16", d=128, C=128, W=128, N=128 * 6 + 40)],
                         ids=["f32", "bf16-C128"])
@pytest.mark.parametrize("how", ["dq_over_lse", "dg_over_lse", "graph"])
def test_backward_on_two_queues(kw, how):
    """The softmax branch runs beside the states and the linear branch.  Results may lie over lse, which its last kernels still
    read when the first results are written; and a captured call replays with both queues.  dq, dk, dv and dg bit for
    bit those of a plain call (the parameter gradients are added atomically: 1e-5 of the largest)."""
    import torch

    w = small("bwd-queues", **dict(dict(Hq=4, Hkv=2, lam=8, B=2), **kw))
    inp = synth.make_inputs(w, seed=201, with_gate=True)
    t = {n: synth.to_torch(inp[n], w.dtype, "cuda") for n in ("q", "k", "v", "g", "Wq", "Wk")}
    dout, out = synth.to_torch(make_dy(w, inp, 202), w.dtype, "cuda"), torch.empty_like(t["q"])
    p = S.make_params(B=w.B, N=w.N, Hq=w.Hq, Hkv=w.Hkv, d=w.d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps,
                      dtype=w.dtype, q=t["q"], k=t["k"], v=t["v"], out=out, g=t["g"])
    sel = torch.zeros(w.B, w.Hq, w.N // w.C, w.lam, dtype=torch.int32, device="cuda")
    ws = torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.still_hybrid_attn_fwd(p, t["q"], t["k"], t["v"], t["g"], t["Wq"], None, t["Wk"], None, out, sel_idx=sel, workspace=ws)
    L = S.still_fwd_workspace_layout(p)
    lse = ws[L.lse:L.lse + w.B * w.Hq * w.N * 4].view(torch.float32).clone()
    bws = torch.empty(S.still_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")

    def grads():
        return {n: torch.zeros_like(t[n[1:]]) for n in ("dq", "dk", "dv", "dg")}, \
               [torch.zeros(w.Hq, w.d, w.d, device="cuda") for _ in range(2)]

    def call(g, dw, l):
        S.still_hybrid_attn_bwd(p, t["q"], t["k"], t["v"], t["g"], t["Wq"], None, t["Wk"], None, out, dout, l, sel,
                                g["dq"], g["dk"], g["dv"], g["dg"], dw[0], None, dw[1], None, bws)

    def check(g, dw):
        for n in g:
            assert torch.equal(g[n], ref[n]), n
        for a_, b_ in zip(dw, dw_ref):
            assert float((a_ - b_).abs().max()) <= 1e-5 * float(b_.abs().max())

    ref, dw_ref = grads()
    call(ref, dw_ref, lse)
    torch.cuda.synchronize()
    assert float(ref["dk"].abs().max()) > 0
    g, dw = grads()
    if how == "graph":
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            call(g, dw, lse)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(g, dw, lse)
        for _ in range(4):
            for x in list(g.values()) + dw:
                x.fill_(7.0)
            bws.fill_(0x5a)
            graph.replay()
            torch.cuda.synchronize()
            check(g, dw)
    else:
        n = how[:2]
        over = g[n].view(torch.uint8).flatten()[:lse.numel() * 4].view(torch.float32)    # the result's own memory
        over.copy_(lse)
        call(g, dw, over)
        torch.cuda.synchronize()
        check(g, dw)


@pytest.mark.parametrize("eager", ["backward", "forward"])
def test_a_call_on_another_stream_stays_out_of_a_capture(eager):
    """A thread that captures a backward pass on one stream may call the library eagerly on another before the capture ends: the
    helper stream is part of the capture then, so the eager call does without it.  Its results are there at once, the
    captured call's after a replay."""
    import torch

    w = small("capture", dtype="bf16", B=2, N=64 * 9 + 5, Hq=4, Hkv=2, lam=8)
    sides = []
    for seed in (231, 232):
        inp = synth.make_inputs(w, seed=seed)
        t = {n: synth.to_torch(inp[n], w.dtype, "cuda") for n in ("q", "k", "v", "Wq", "Wk")}
        t["dout"], t["out"] = synth.to_torch(make_dy(w, inp, seed + 10), w.dtype, "cuda"), torch.empty_like(t["q"])
        p = S.make_params(B=w.B, N=w.N, Hq=w.Hq, Hkv=w.Hkv, d=w.d, C=w.C, W=w.W, lam=w.lam, scale=w.scale, eps=w.eps,
                          dtype=w.dtype, q=t["q"], k=t["k"], v=t["v"], out=t["out"])
        t.update(sel=torch.zeros(w.B, w.Hq, w.N // w.C, w.lam, dtype=torch.int32, device="cuda"),
                 ws=torch.empty(S.still_fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda"),
                 bws=torch.empty(S.still_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda"),
                 dW=[torch.zeros(w.Hq, w.d, w.d, device="cuda") for _ in range(2)])
        t.update({"d" + n: torch.zeros_like(t[n]) for n in ("q", "k", "v")})
        L = S.still_fwd_workspace_layout(p)
        t["lse"] = t["ws"][L.lse:L.lse + w.B * w.Hq * w.N * 4].view(torch.float32)
        sides.append((p, t))

    def forward(p, t, stream):
        S.still_hybrid_attn_fwd(p, t["q"], t["k"], t["v"], None, t["Wq"], None, t["Wk"], None, t["out"], sel_idx=t["sel"],
                                workspace=t["ws"], stream=stream)

    def backward(p, t, stream):
        S.still_hybrid_attn_bwd(p, t["q"], t["k"], t["v"], None, t["Wq"], None, t["Wk"], None, t["out"], t["dout"], t["lse"], t["sel"],
                                t["dq"], t["dk"], t["dv"], None, t["dW"][0], None, t["dW"][1], None, t["bws"], stream=stream)

    names = {"backward": ("dq", "dk", "dv"), "forward": ("out",)}
    ref = []
    for p, t in sides:
        for call in (forward, backward):
            call(p, t, torch.cuda.current_stream())
        torch.cuda.synchronize()
        ref.append({n: t[n].clone() for n in ("dq", "dk", "dv", "out")})
        for n in names["backward"]:
            t[n].fill_(7.0)
    if eager == "forward":
        sides[1][1]["out"].fill_(7.0)
    torch.cuda.synchronize()
    one, two, graph = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=one):
        backward(*sides[0], one)
        (backward if eager == "backward" else forward)(*sides[1], two)
    torch.cuda.synchronize()
    for n in names[eager]:
        assert torch.equal(sides[1][1][n], ref[1][n]), n
    for n in names["backward"]:
        assert bool((sides[0][1][n] == 7.0).all()), n            # captured, not run
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        for n in names["backward"]:
            assert torch.equal(sides[0][1][n], ref[0][n]), n
            sides[0][1][n].fill_(7.0)

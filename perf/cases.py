"""The work that a user of the d2Cache step library has it do, as timed cases.

Every case goes through the public entry points of paper_2509_23094_amd.binding (the same names as include/d2c.h):

  step       d2c_step: one denoising step of a whole model.  First steps (every row selected; the sequence was
             just reset), decode steps in the middle of a generation, one sequence or several in one group.
  layer      d2c_refresh_layer over a stack of blocks, as a program does that drives the partial forward itself
             (own hidden rows, own caches), with the rollout block and d2c_influence behind it or without them.
  attention  d2c_attention: the selected queries against the whole cache, with or without the head average.
  linear     d2c_linear: one projection on a ragged handful of rows, row-major weights (the vocabulary head, or
             a matrix of a block).
  select     d2c_select: Eq. 1 on some logit rows and the two-stage selection.

Geometries are those of paper_2509_23094_amd.workloads: C3 / C5 (LLaDA-8B shape), C4 / C6 (Dream-7B shape) in bf16
and C1, the small fp32 model.  Inputs are random with the distributions of workloads.py (weights N(0, 0.02), so that
cached K and V rows have a standard deviation of 0.02 sqrt(d_model)), drawn on the device from the seed.
"""
import math
from dataclasses import replace

import numpy as np
import torch

from paper_2509_23094_amd import binding as B
from paper_2509_23094_amd import workloads as W

# What a decode step selects besides the masked tokens of its block and the token decoded last: the top-p stage
# takes about this share of the known tokens (p = 0.1 of a mildly uneven influence vector).
U_SHARE = 0.075


def listed():
    return [
        # Whole steps have full width and vocabulary and a quarter of the depth: rounding grows from block to block, and
        # two correct implementations of 32 blocks in bf16 are too far apart (about 3 %) to be told from a wrong one.
        # The decode step of the benchmark: LLaDA-8B shape, prompt 256 + 256 generated, middle of a block
        dict(name="step llada decode", kind="step", model="C3", layers=8, batch=1, prompt=256, gen=256, block=32,
             unmask=1, done=112, first=False),
        # the first step of the same generation: every row, fills the caches, head on all masked rows
        dict(name="step llada first", kind="step", model="C3", layers=8, batch=1, prompt=256, gen=256, block=32,
             unmask=1, done=0, first=True),
        # Dream-7B shape (GQA 28/4, vocabulary 152064), an odd length, late in the generation
        dict(name="step dream decode", kind="step", model="C4", layers=8, batch=1, prompt=509, gen=256, block=32,
             unmask=1, done=181, first=False),
        # serving a batch of long sequences: four sequences of 3072 positions, two tokens a step
        dict(name="step llada batch long", kind="step", model="C3", layers=8, batch=4, prompt=2048, gen=1024, block=64,
             unmask=2, done=420, first=False),
        # a program that drives the blocks itself: long Dream-shaped generation, odd sizes, rollout kept
        dict(name="layers dream long", kind="layer", model="C4", layers=2, L=1823, m=97, rollout=True),
        # every row of an odd-length LLaDA-shaped sequence, no rollout wanted (filling the caches)
        dict(name="layers llada all rows", kind="layer", model="C3", layers=2, L=777, m=777, rollout=False),
        # the small fp32 model: launches and latency
        dict(name="layers small f32", kind="layer", model="C1", layers=2, L=128, m=37, rollout=True),
        # the isolated attention op of the benchmark
        dict(name="attention llada 256", kind="attention", model="C3", L=2048, m=256, average=True, refresh=True),
        # a handful of GQA queries against an odd cache length, output only
        dict(name="attention dream few", kind="attention", model="C4", L=1023, m=33, average=False, refresh=True),
        # the vocabulary head on the masked rows of a block
        dict(name="linear llada head", kind="linear", model="C3", L=512, m=17, n_out=126464, k_in=4096),
        # the selection of a short generation: the smallest call of the serving loop
        dict(name="select short", kind="select", vocab=126464, L=512, prompt=256, rows=16, k=32, p=0.1, block=32,
             unmask=1, known=0.4),
        # the selection of a first step at the Dream vocabulary, fully non-autoregressive, long sequence
        dict(name="select long", kind="select", vocab=152064, L=3071, prompt=2048, rows=200, k=32, p=0.1, block=1024,
             unmask=2, known=0.3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "layer", "layer", "attention", "attention", "linear", "select"])
    if kind == "step":
        model = rng.choice(["C3", "C4"])
        first = rng.random() < 0.3
        batch = rng.choice([1, 1, 2, 3, 4])
        prompt, gen = _log(rng, 32, 2048), _log(rng, 64, 1024)
        # whole-width models of reduced depth, as the tests take them; no more rows x layers than the long batch has
        layers = rng.randint(2, 6)
        while first and layers * batch * (prompt + gen) > 6000:
            batch, prompt, gen = max(1, batch - 1), max(32, prompt // 2), max(64, gen // 2)
        unmask = rng.choice([1, 1, 2, 4])
        block = rng.choice([16, 32, 64])
        done = 0 if first else rng.randint(unmask, gen - 8)
        return dict(kind="step", model=model, layers=layers, batch=batch, prompt=prompt, gen=gen, block=block,
                    unmask=unmask, done=done, first=first)
    if kind == "layer":
        model = rng.choice(["C3", "C4", "C3", "C4", "C1"])
        L = _log(rng, 64, 1024 if model == "C1" else 3072)
        m = L if rng.random() < 0.2 else min(L, _log(rng, 1, 1024))
        rollout = rng.random() < 0.7
        if rollout and model != "C1":
            m = min(m, 1024)
        return dict(kind="layer", model=model, layers=rng.randint(1, 2), L=L, m=m, rollout=rollout)
    if kind == "attention":
        model = rng.choice(["C3", "C4", "C3", "C4", "C1"])
        L = _log(rng, 48, 1024 if model == "C1" else 4096)
        return dict(kind="attention", model=model, L=L, m=min(L, _log(rng, 1, 1024)), average=rng.random() < 0.6,
                    refresh=rng.random() < 0.8)
    if kind == "linear":
        model = rng.choice(["C3", "C4", "C3", "C4", "C1"])
        d = W.DIMS[model]
        n_out, k_in = rng.choice([(d.d_q + 2 * d.d_kv, d.d_model), (d.d_model, d.d_q), (2 * d.d_ffn, d.d_model),
                                  (d.d_model, d.d_ffn), (d.vocab, d.d_model)])
        return dict(kind="linear", model=model, L=1024, m=_log(rng, 1, 256 if n_out == d.vocab else 1024),
                    n_out=n_out, k_in=k_in)
    L = _log(rng, 64, 4096)
    prompt = rng.randint(L // 4, 3 * L // 4)
    block = rng.choice([16, 32, 64, L - prompt])
    return dict(kind="select", vocab=rng.choice([126464, 152064]), L=L, prompt=prompt,
                rows=min(_log(rng, 1, 256), max(1, (L - prompt) // 3)), k=rng.choice([8, 32, 64]),
                p=rng.choice([0.05, 0.1, 0.3]), block=block, unmask=rng.choice([1, 2]), known=rng.uniform(0.05, 0.6))


# ---------------------------------------------------------------------------------------------- inputs from the seed
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def _dtype(dims):
    return torch.bfloat16 if dims.dtype == "bf16" else torch.float32


def _gain(g, n):
    return 1.0 + _normal(g, (n,), 0.1, torch.float32)


def _weights(g, dims, vocab):
    t = _dtype(dims)
    d, f = dims.d_model, dims.d_ffn
    layers = [{"attn_norm": _gain(g, d), "wqkv": _normal(g, (dims.d_q + 2 * dims.d_kv, d), 0.02, t),
               "wo": _normal(g, (d, dims.d_q), 0.02, t), "ffn_norm": _gain(g, d),
               "w_gate_up": _normal(g, (2 * f, d), 0.02, t), "w_down": _normal(g, (d, f), 0.02, t)}
              for _ in range(dims.n_layers)]
    return {"tok_emb": _normal(g, (vocab, d), 0.02, t), "final_norm": _gain(g, d),
            "lm_head": _normal(g, (vocab, d), 0.02, t), "layers": layers}


def _rows(rng, L, m):
    return np.sort(rng.choice(L, size=m, replace=False)).astype(np.int32)


def _step_shape(case, rng):
    """One sequence in the middle of its generation: masked flags, S_t and the compact rows that are still masked."""
    P, G, blk = case["prompt"], case["gen"], case["block"]
    L = P + G
    masked = np.zeros(L, np.uint8)
    masked[P:] = 1
    if case["first"]:
        return masked, np.arange(L, dtype=np.int32), np.flatnonzero(masked).astype(np.int32)
    done = case["done"]
    full = P + (done // blk) * blk                                     # whole blocks in front of the current one
    masked[P:full] = 0
    hi = min(L, full + blk)
    masked[rng.choice(np.arange(full, hi), size=min(done % blk, hi - full - 1), replace=False)] = 0
    known = np.flatnonzero(masked == 0)
    take = {int(i) for i in np.flatnonzero(masked[:hi])[:32]}          # M*, k = 32
    fresh = known[-case["unmask"]:]                                    # decoded by the step before
    u = rng.choice(known[:-case["unmask"]], size=max(1, int(round(U_SHARE * len(known)))), replace=False)
    s = np.array(sorted(take | {int(i) for i in fresh} | {int(i) for i in u}), np.int32)
    return masked, s, np.flatnonzero(masked[s]).astype(np.int32)


def _step_inputs(case, seed):
    dims = W.with_layers(W.DIMS[case["model"]], case["layers"])
    g, rng = _gen(seed), np.random.default_rng([int(seed), 1])
    L = case["prompt"] + case["gen"]
    weights = _weights(g, dims, dims.vocab)
    std = 0.02 * math.sqrt(dims.d_model)
    seqs = []
    for _ in range(case["batch"]):
        masked, s, rows = _step_shape(case, rng)
        tokens = rng.integers(0, dims.vocab - 1, size=L).astype(np.int32)
        tokens[masked != 0] = dims.mask_id
        shape = (dims.n_layers, L, dims.d_kv)
        if case["first"]:
            kc = vc = None
        else:
            kc, vc = _normal(g, shape, std, _dtype(dims)), _normal(g, shape, std, _dtype(dims))
        conf = (rng.random(L) * 2e-3 * (masked != 0)).astype(np.float32)
        pred = rng.integers(0, dims.vocab - 1, size=L).astype(np.int32)
        seqs.append(dict(tokens=tokens, masked=masked, s=s, rows=rows, k=kc, v=vc, conf=conf, pred=pred))
    return dims, weights, seqs


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _prepare_step(case, seed):
    dims, weights, seqs = _step_inputs(case, seed)
    L = case["prompt"] + case["gen"]
    ctx = B.Context(dims, weights, L, device_weights=True, max_batch=case["batch"])
    prm = B.make_params(10.0, 32, 0.1, case["block"], case["unmask"])
    st = dict(case=case, ctx=ctx, prm=prm, seqs=[], keep=[])
    for q in seqs:
        seq = B.Sequence_(ctx, q["tokens"], q["masked"], case["prompt"], trace=True, max_trace_rows=max(1, len(q["rows"])))
        if not case["first"]:
            seq.k_cache.copy_(q["k"])
            seq.v_cache.copy_(q["v"])
            seq.conf.copy_(_dev(q["conf"]))
            seq.pred.copy_(_dev(q["pred"]))
            seq.set_selection(q["s"], q["rows"])
        st["seqs"].append(seq)
        st["keep"].append(dict(tokens=seq.tokens.clone(), masked=seq.is_masked.clone(), s=seq.s_idx.clone(),
                               rows=seq.s_rows.clone(), n_s=len(q["s"]), n_rows=len(q["rows"]),
                               n_masked=int(q["masked"].sum())))
    return st


def _run_step(st):
    # the step decodes in place: the sequence is put back to where it stood (as a program does that starts a
    # generation, or takes a step again from a saved state)
    first = st["case"]["first"]
    for seq, keep in zip(st["seqs"], st["keep"]):
        seq.tokens.copy_(keep["tokens"])
        seq.is_masked.copy_(keep["masked"])
        if first:
            st["ctx"].d2c_seq_reset(seq)
        else:
            seq.s_idx.copy_(keep["s"])
            seq.s_rows.copy_(keep["rows"])
            seq.c.n_s, seq.c.n_rows, seq.c.n_masked = keep["n_s"], keep["n_rows"], keep["n_masked"]
    st["ctx"].d2c_step(st["prm"], st["seqs"])
    # The selected sets are not compared here: random weights give a nearly flat influence vector, so the cut of the
    # top-p stage is decided by rounding.  The influence itself is, and the select cases compare the sets exactly.
    return [{"logits": s.logits_out[: k["n_rows"]], "hidden": s.hidden_out[: k["n_s"]], "k": s.k_cache, "v": s.v_cache,
             "conf": s.conf, "influence": s.influence, "tokens": s.tokens, "is_masked": s.is_masked}
            for s, k in zip(st["seqs"], st["keep"])]


def _layer_inputs(case, seed):
    dims = W.with_layers(W.DIMS[case["model"]], case["layers"])
    g, rng = _gen(seed), np.random.default_rng([int(seed), 2])
    L, m = case["L"], case["m"]
    weights = _weights(g, dims, dims.vocab if case["model"] == "C1" else 1024)        # the head is not reached
    std = 0.02 * math.sqrt(dims.d_model)
    t = _dtype(dims)
    kc = _normal(g, (dims.n_layers, L, dims.d_kv), std, t)
    vc = _normal(g, (dims.n_layers, L, dims.d_kv), std, t)
    h0 = _normal(g, (m, dims.d_model), 0.5, torch.float32)
    return dims, weights, kc, vc, h0, _rows(rng, L, m)


def _prepare_layer(case, seed):
    dims, weights, kc, vc, h0, idx = _layer_inputs(case, seed)
    vocab = weights["tok_emb"].shape[0]
    small = dims if vocab == dims.vocab else replace(dims, vocab=vocab)
    ctx = B.Context(small, weights, case["L"], device_weights=True)
    st = dict(case=case, ctx=ctx, h0=h0, h=torch.empty_like(h0), k=kc, v=vc, idx=_dev(idx), idx_host=idx, avg=None, roll=None)
    if case["rollout"]:
        st["avg"] = torch.empty((case["m"], case["L"]), dtype=torch.float32, device="cuda")
        st["roll"] = torch.empty_like(st["avg"])
        st["c"] = torch.empty(case["L"], dtype=torch.float32, device="cuda")
    return st


def _run_layer(st):
    ctx, L = st["ctx"], st["case"]["L"]
    st["h"].copy_(st["h0"])                                             # the blocks work in place on the hidden rows
    for l in range(st["case"]["layers"]):
        ctx.d2c_refresh_layer(l, st["h"], st["idx"], st["idx_host"], st["k"][l], st["v"][l], L, st["avg"], st["roll"])
    out = {"hidden": st["h"], "k": st["k"], "v": st["v"]}
    if st["roll"] is not None:
        ctx.d2c_influence(st["roll"], st["idx"], len(st["idx_host"]), L, st["c"])
        out.update(average=st["avg"], rollout=st["roll"], influence=st["c"])
    return out


def _attention_inputs(case, seed):
    dims = W.DIMS[case["model"]]
    g, rng = _gen(seed), np.random.default_rng([int(seed), 3])
    L, m, t = case["L"], case["m"], _dtype(dims)
    q = _normal(g, (m, dims.d_q), 1.0, t)
    kc, vc = _normal(g, (L, dims.d_kv), 1.0, t), _normal(g, (L, dims.d_kv), 1.0, t)
    nk, nv = _normal(g, (m, dims.d_kv), 1.0, t), _normal(g, (m, dims.d_kv), 1.0, t)
    return dims, q, kc, vc, nk, nv, _rows(rng, L, m)


def _prepare_attention(case, seed):
    dims, q, kc, vc, nk, nv, idx = _attention_inputs(case, seed)
    wd = W.ModelDims(1, dims.d_q, dims.n_heads, dims.n_kv_heads, dims.head_dim, 64, 64, dtype=dims.dtype)
    ctx = B.Context(wd, _weights(_gen(seed + 1), wd, 64), case["L"], device_weights=True)
    if not case["refresh"]:
        nk = nv = None
    avg = torch.empty((case["m"], case["L"]), dtype=torch.float32, device="cuda") if case["average"] else None
    return dict(case=case, ctx=ctx, q=q, k=kc, v=vc, nk=nk, nv=nv, idx=_dev(idx), out=torch.empty_like(q), avg=avg)


def _run_attention(st):
    c = st["case"]
    st["ctx"].d2c_attention(st["q"], st["idx"], c["m"], st["nk"], st["nv"], st["k"], st["v"], c["L"], st["out"], st["avg"])
    out = {"out": st["out"], "k": st["k"], "v": st["v"]}
    if st["avg"] is not None:
        out["average"] = st["avg"]
    return out


def _linear_inputs(case, seed):
    dims = W.DIMS[case["model"]]
    g, t = _gen(seed), _dtype(dims)
    return dims, _normal(g, (case["m"], case["k_in"]), 1.0, t), _normal(g, (case["n_out"], case["k_in"]), 0.02, t)


def _prepare_linear(case, seed):
    dims, a, w = _linear_inputs(case, seed)
    wd = replace(W.with_layers(dims, 1), vocab=1024)
    ctx = B.Context(wd, _weights(_gen(seed + 1), wd, 1024), case["L"], device_weights=True)
    return dict(case=case, ctx=ctx, a=a, w=w, out=torch.empty((case["m"], case["n_out"]), dtype=torch.float32, device="cuda"))


def _run_linear(st):
    c = st["case"]
    st["ctx"].d2c_linear(st["a"], st["w"], c["m"], c["n_out"], c["k_in"], st["out"])
    return st["out"]


def _select_inputs(case, seed):
    g, rng = _gen(seed), np.random.default_rng([int(seed), 4])
    L, P, V = case["L"], case["prompt"], case["vocab"]
    masked = np.zeros(L, np.uint8)
    masked[P:] = rng.random(L - P) >= case["known"]
    masked[P + int(rng.integers(0, L - P))] = 1
    at = np.flatnonzero(masked)[: case["rows"]].astype(np.int32)
    logits = _normal(g, (len(at), V), 2.0, torch.float32)
    tokens = rng.integers(0, V - 1, size=L).astype(np.int32)
    tokens[masked != 0] = V - 1
    conf = (rng.random(L) ** 8).astype(np.float32)                       # a few confident rows
    c = 1.0 / (1.0 + rng.permutation(L))                                 # a Zipf tail and a few sinks
    c[rng.choice(L, size=4, replace=False)] += 0.125 * L
    influence = (c * (L / c.sum())).astype(np.float32)
    return logits, at, tokens, masked, conf, rng.integers(0, V - 1, size=L).astype(np.int32), influence


def _prepare_select(case, seed):
    logits, at, tokens, masked, conf, pred, influence = _select_inputs(case, seed)
    L, V = case["L"], case["vocab"]
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")                # the selection reads no weight
    weights = _weights(_gen(seed + 1), wd, 64)
    weights["tok_emb"] = weights["lm_head"] = torch.zeros((V, 64), dtype=torch.float32, device="cuda")
    ctx = B.Context(wd, weights, L, device_weights=True)
    st = dict(case=case, ctx=ctx, prm=B.make_params(10.0, case["k"], case["p"], case["block"], case["unmask"]), logits=logits,
              at=_dev(at), tokens0=_dev(tokens), masked0=_dev(masked), tokens=_dev(tokens), masked=_dev(masked), conf=_dev(conf),
              pred=_dev(pred), influence=_dev(influence), score=torch.zeros(L, dtype=torch.float32, device="cuda"),
              counts=torch.zeros(B.N_COUNTS, dtype=torch.int32, device="cuda"))
    for name in ("mstar", "u", "decode", "s", "s_rows"):
        st[name] = torch.full((L,), -1, dtype=torch.int32, device="cuda")
    return st


def _run_select(st):
    st["tokens"].copy_(st["tokens0"])                                   # the call unmasks in place
    st["masked"].copy_(st["masked0"])
    st["ctx"].d2c_select(st["prm"], st["logits"], st["at"], len(st["at"]), st["tokens"], st["masked"], st["case"]["L"],
                         st["case"]["prompt"], st["conf"], st["pred"], st["influence"], st["mstar"], st["u"], st["decode"],
                         st["s"], st["s_rows"], st["counts"], st["score"])
    return {k: st[k] for k in ("tokens", "masked", "conf", "pred", "mstar", "u", "decode", "s", "s_rows", "counts", "score")}


def prepare(case, seed):
    return {"step": _prepare_step, "layer": _prepare_layer, "attention": _prepare_attention, "linear": _prepare_linear,
            "select": _prepare_select}[case["kind"]](case, int(seed))


def run(state):
    return {"step": _run_step, "layer": _run_layer, "attention": _run_attention, "linear": _run_linear,
            "select": _run_select}[state["case"]["kind"]](state)


# ---------------------------------------------------------------------------------------------- what a pass has to do
def _block_work(dims, m, keys, seqs=1):
    """Bytes and operations of one block on m rows in all, against `keys` cached positions in all: weights and K/V
    once, the hidden rows in and out, the new K/V rows out."""
    ts = 2 if dims.dtype == "bf16" else 4
    w = (dims.d_q + 2 * dims.d_kv) * dims.d_model + dims.d_model * dims.d_q + 3 * dims.d_model * dims.d_ffn
    by = w * ts + 2 * keys * dims.d_kv * ts + 2 * m * dims.d_kv * ts
    fl = 2.0 * m * w + 4.0 * (m / seqs) * keys * dims.d_q
    return by, fl


def work(case):
    kind = case["kind"]
    if kind == "step":
        dims, b = W.with_layers(W.DIMS[case["model"]], case["layers"]), case["batch"]
        L = case["prompt"] + case["gen"]
        _, s, rows = _step_shape(case, np.random.default_rng([0, 1]))
        m, n = len(s) * b, len(rows) * b
        by, fl = _block_work(dims, m, L * b, b)
        by, fl = by * case["layers"], fl * case["layers"]
        by += dims.vocab * dims.d_model * 2 + n * dims.vocab * 4 + m * dims.d_model * (2 + 4)
        fl += 2.0 * n * dims.vocab * dims.d_model + 2.0 * case["layers"] * m * L
        return {"bytes": by, "flops": fl}
    if kind == "layer":
        dims = W.DIMS[case["model"]]
        m, L, n = case["m"], case["L"], case["layers"]
        by, fl = _block_work(dims, m, L)
        by, fl = by * n + 2 * m * dims.d_model * 4, fl * n
        if case["rollout"]:
            by += 4 * m * L * (n + 1)
            fl += 2.0 * m * m * L * (n - 1)
        return {"bytes": by, "flops": fl}
    if kind == "attention":
        dims = W.DIMS[case["model"]]
        ts = 2 if dims.dtype == "bf16" else 4
        m, L = case["m"], case["L"]
        by = 2 * L * dims.d_kv * ts + 2 * m * dims.d_q * ts
        by += 2 * 2 * m * dims.d_kv * ts if case["refresh"] else 0
        by += 4 * m * L if case["average"] else 0
        return {"bytes": by, "flops": 4.0 * m * L * dims.d_q}
    if kind == "linear":
        ts = 2 if W.DIMS[case["model"]].dtype == "bf16" else 4
        m, n, k = case["m"], case["n_out"], case["k_in"]
        return {"bytes": (m + n) * k * ts + 4 * m * n, "flops": 2.0 * m * n * k}
    rows = case["rows"]
    return {"bytes": rows * case["vocab"] * 4 + case["L"] * 45, "flops": 3.0 * rows * case["vocab"]}


# ---------------------------------------------------------------------------------------------- tolerances
def tolerance(case):
    kind = case["kind"]
    f32 = kind == "select" or W.DIMS[case.get("model", "C1")].dtype == "f32"
    if kind == "select":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    if f32:
        return {"rel": 1e-5, "max": 1e-3}
    if kind == "linear":
        return {"rel": 1e-5, "max": 1e-4}                                # bf16 operands, sums and results in 32 bits
    if kind == "attention":
        return {"rel": 1e-2, "max": 0.05}
    if kind == "layer":
        return {"rel": 2e-2, "max": 0.15}                                # other summation orders were seen to give 0.5 %
    return {"rel": 3e-2, "max": 0.5, "differ": 0.01}                     # as above over eight blocks: 1 %


# ---------------------------------------------------------------------------------------------- the same in 64 bits
F = torch.float64


def _norm64(h, gain, eps):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + eps) * gain.to(F)


def _mm64(a, w):
    """a [m, K] times w[N, K] transposed; the weight is widened a slab at a time."""
    return torch.cat([a @ part.to(F).t() for part in w.split(16384)], dim=1)


def _rope64(x, pos, theta):
    half = x.shape[-1] // 2
    ang = pos.to(F)[:, None] * (float(theta) ** (-torch.arange(half, dtype=F, device="cuda") / half))[None, :]
    cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)


def _attend64(dims, q, k, v):
    """q [m, H dh], k and v [L, Hkv dh]: output and the mean over heads of the softmax rows."""
    m, L, dh, grp = q.shape[0], k.shape[0], dims.head_dim, dims.n_heads // dims.n_kv_heads
    out = torch.empty((m, dims.d_q), dtype=F, device="cuda")
    avg = torch.zeros((m, L), dtype=F, device="cuda")
    for h in range(dims.n_heads):
        g = h // grp
        p = torch.softmax(q[:, h * dh:(h + 1) * dh] @ k[:, g * dh:(g + 1) * dh].t() / math.sqrt(dh), dim=-1)
        out[:, h * dh:(h + 1) * dh] = p @ v[:, g * dh:(g + 1) * dh]
        avg += p
    return out, avg / dims.n_heads


def _block64(dims, w, h, idxs, caches):
    """One block on the rows of several sequences; caches: (k, v) in 64 bits per sequence, updated in place."""
    n = h.shape[0]
    qkv = _mm64(_norm64(h, w["attn_norm"], dims.rms_eps), w["wqkv"])
    q, k, v = qkv.split([dims.d_q, dims.d_kv, dims.d_kv], dim=1)
    outs, avgs, off = [], [], 0
    for idx, (kc, vc) in zip(idxs, caches):
        part = slice(off, off + len(idx))
        off += len(idx)
        kc[idx] = _rope64(k[part].reshape(-1, dims.n_kv_heads, dims.head_dim), idx, dims.rope_theta).reshape(len(idx), -1)
        vc[idx] = v[part]
        qs = _rope64(q[part].reshape(-1, dims.n_heads, dims.head_dim), idx, dims.rope_theta).reshape(len(idx), -1)
        o, a = _attend64(dims, qs, kc, vc)
        outs.append(o)
        avgs.append(a)
    assert off == n
    h = h + _mm64(torch.cat(outs), w["wo"])
    gu = _mm64(_norm64(h, w["ffn_norm"], dims.rms_eps), w["w_gate_up"])
    gate, up = gu.chunk(2, dim=1)
    return h + _mm64(torch.nn.functional.silu(gate) * up, w["w_down"]), avgs


def _exact_step(case, seed):
    dims, weights, seqs = _step_inputs(case, seed)
    L = case["prompt"] + case["gen"]
    idxs = [_dev(q["s"]).long() for q in seqs]
    h = torch.cat([weights["tok_emb"][_dev(q["tokens"]).long()[i]] for q, i in zip(seqs, idxs)]).to(F)
    new = [([], []) for _ in seqs]
    infl = []
    avgs = [[] for _ in seqs]
    for l, w in enumerate(weights["layers"]):
        caches = []
        for q in seqs:
            if q["k"] is None:
                caches.append(tuple(torch.zeros((L, dims.d_kv), dtype=F, device="cuda") for _ in range(2)))
            else:
                caches.append((q["k"][l].to(F), q["v"][l].to(F)))
        h, a = _block64(dims, w, h, idxs, caches)
        for i, (kc, vc) in enumerate(caches):
            new[i][0].append(kc.float())                                # 24 bits are enough to compare 8 with
            new[i][1].append(vc.float())
            avgs[i].append(a[i])
    for idx, mine in zip(idxs, avgs):
        v = torch.ones(L, dtype=F, device="cuda")
        outside = torch.ones(L, dtype=F, device="cuda")
        outside[idx] = 0.0
        for a in reversed(mine):
            v = 0.5 * (v[idx] @ a + (outside + 1.0) * v)
        infl.append(v)
    got, off = [], 0
    for i, q in enumerate(seqs):
        mine = h[off: off + len(q["s"])]
        off += len(q["s"])
        rows = _dev(q["rows"]).long()
        logits = _mm64(_norm64(mine[rows], weights["final_norm"], dims.rms_eps), weights["lm_head"])
        # the confidences are a dozen numbers that the logits fix: how far they are off is luck, so the logits stand for them
        got.append({"logits": logits, "hidden": mine, "k": torch.stack(new[i][0]), "v": torch.stack(new[i][1]), "conf": None,
                    "influence": infl[i], "tokens": None, "is_masked": None})
    return got


def _exact_layer(case, seed):
    dims, weights, kc, vc, h, idx = _layer_inputs(case, seed)
    L, at = case["L"], _dev(idx).long()
    h, kc, vc = h.to(F), kc.to(F), vc.to(F)
    roll = torch.zeros((case["m"], L), dtype=F, device="cuda")
    roll[torch.arange(case["m"], device="cuda"), at] = 1.0
    outside = torch.ones(L, dtype=F, device="cuda")
    outside[at] = 0.0
    for l, w in enumerate(weights["layers"]):
        h, (avg,) = _block64(dims, w, h, [at], [(kc[l], vc[l])])
        if case["rollout"]:
            roll = 0.5 * (avg[:, at] @ roll + avg * outside + roll)
    out = {"hidden": h, "k": kc, "v": vc}
    if case["rollout"]:
        out.update(average=avg, rollout=roll, influence=outside + roll.sum(0))
    return out


def _exact_attention(case, seed):
    dims, q, kc, vc, nk, nv, idx = _attention_inputs(case, seed)
    kc, vc = kc.to(F), vc.to(F)
    if case["refresh"]:
        at = _dev(idx).long()
        kc[at], vc[at] = nk.to(F), nv.to(F)
    o, a = _attend64(dims, q.to(F), kc, vc)
    out = {"out": o, "k": kc, "v": vc}
    if case["average"]:
        out["average"] = a
    return out


def _exact_linear(case, seed):
    _, a, w = _linear_inputs(case, seed)
    return _mm64(a.to(F), w)


def _exact_select(case, seed):
    logits, at, tokens, masked, conf, pred, influence = _select_inputs(case, seed)
    L = case["L"]
    where = _dev(at).long()
    x = logits.to(F)
    conf = _dev(conf).to(F)
    conf[where] = torch.exp(x.max(dim=1).values - torch.logsumexp(x, dim=1))
    first = int(np.flatnonzero(masked)[0])
    lo = case["prompt"] + (first - case["prompt"]) // case["block"] * case["block"]
    hi = min(L, lo + case["block"])
    pos = torch.arange(L, dtype=F, device="cuda")
    phi = torch.exp(-((pos[:, None] - pos[None, :]) ** 2) / (2.0 * 10.0 ** 2))
    density = phi @ (_dev(masked) == 0).to(F)
    score = torch.zeros(L, dtype=F, device="cuda")
    here = torch.from_numpy(np.flatnonzero(masked[lo:hi]) + lo).cuda()
    score[here] = density[here] * conf[here]
    got = {k: None for k in ("tokens", "masked", "pred", "mstar", "u", "decode", "s", "s_rows", "counts")}
    return dict(got, conf=conf, score=score)


def exact(case, seed):
    return {"step": _exact_step, "layer": _exact_layer, "attention": _exact_attention, "linear": _exact_linear,
            "select": _exact_select}[case["kind"]](case, int(seed))

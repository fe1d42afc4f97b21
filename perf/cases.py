"""The work that is timed: calls of the public entry points of paper_2402_11809_amd, at the sizes that its
shapes, tests and benchmark use.

Four kinds of call:
  step     Model.step: one auto-correct step (forward over the block, verification, next block) against a
           cache of given lengths.  The commit behind it is one launch of a few integers and is left out, so
           that a pass can be repeated on the same state.
  prefill  Model.prefill: one prompt chunk against a cache that may already hold earlier chunks.
  sample   Model.sample_verify: the verification by rejection sampling on a step's logits.
  loss     Model.sar_loss: the loss reduction of the finetuning half.

Weights are N(0, 0.02) and cached keys / values N(0, 1), both bf16, as in the repository's benchmark; all of
it is drawn on the GPU from the seed alone.  Most cases run one to four layers of a model's width; one runs
all 32 layers of the 7B shape.
"""
from __future__ import annotations

import gc
import math
from dataclasses import dataclass

import numpy as np
import torch

from paper_2402_11809_amd import binding, layout
from space_inputs import SHAPES, ModelShape

# A model of which only the vocabulary matters: sample and loss calls read logits and nothing else.
HEAD_ONLY = ModelShape("head-only", 1, 256, 4, 64, 688, 32000)
DEV = "cuda:0"


# ------------------------------------------------------------------------------------------- the cases

def listed():
    return [
        # A small model with a short prompt: nothing but launches and latencies.
        dict(name="step_tiny_k4", kind="step", shape="tiny", layers=2, k=4, ctx="96", paged=False, tuned=False),
        # The decoding step at the benchmark's width and context (two layers and the head).
        dict(name="step_7b_2l_k5", kind="step", shape="7b", layers=2, k=5, ctx="518", paged=False, tuned=False),
        # ... and the whole model: the latency of one step of a lone request.
        dict(name="step_7b_32l_k5", kind="step", shape="7b", layers=32, k=5, ctx="527", paged=False, tuned=False),
        # A longer context, where the keys of a head no longer pass through one compute unit.
        dict(name="step_13b_2l_k5_long", kind="step", shape="13b", layers=2, k=5, ctx="2047", paged=False, tuned=False),
        # The widest member of the family: eight query heads to a key/value head.
        dict(name="step_70b_1l_k5", kind="step", shape="70b", layers=1, k=5, ctx="1023", paged=False, tuned=False),
        # Serving: eight requests of ragged lengths over the paged cache, as the continuous batcher runs them.
        dict(name="step_7b_2l_b8_k5_paged", kind="step", shape="7b", layers=2, k=5,
             ctx="261,417,733,1010,1484,2290,3071,3999", paged=True, tuned=True),
        # The widest block the benchmark batches: 648 rows, bound by the matrix unit.
        dict(name="step_7b_2l_b8_k8", kind="step", shape="7b", layers=2, k=8,
             ctx="458,611,902,1377,1795,2204,2901,3685", paged=False, tuned=True),
        # A full prompt chunk behind an earlier one (a prompt of 2048 tokens in two chunks).
        dict(name="prefill_7b_4l_1024", kind="prefill", shape="7b", layers=4, rows=1024, ctx="1024", paged=False, tuned=True),
        # A short prompt of odd length into an empty cache.
        dict(name="prefill_7b_4l_333", kind="prefill", shape="7b", layers=4, rows=333, ctx="0", paged=False, tuned=False),
        # Sampling instead of greedy verification: a lone request with the paper's top-k and top-p ...
        dict(name="sample_b1_k5", kind="sample", batch=1, k=5, top_k=10, top_p=0.95, residual=True),
        # ... and a batch with a long list of kept tokens.
        dict(name="sample_b8_k8", kind="sample", batch=8, k=8, top_k=50, top_p=0.95, residual=False),
        # The loss of one finetuning sequence, prompt rows ignored.
        dict(name="loss_2048", kind="loss", rows=2048, vocab=32000),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["prefill"] * 3 + ["sample"] * 2 + ["loss"])
    if kind == "loss":
        return dict(kind=kind, rows=_log_int(rng, 40, 3000), vocab=rng.choice([1000, 32000]))
    if kind == "sample":
        batch, k = rng.randint(1, 8), rng.randint(1, 8)
        return dict(kind=kind, batch=batch, k=k, top_k=_log_int(rng, 2, 64), top_p=rng.choice([0.5, 0.9, 0.95, 1.0]),
                    residual=rng.random() < 0.5)
    shape = rng.choice(["tiny", "small128", "gqa128", "7b", "7b", "7b", "13b", "70b"])
    layers = 1 if shape == "70b" else rng.randint(1, 2)
    if kind == "prefill":
        return dict(kind=kind, shape=shape, layers=layers + 1, rows=_log_int(rng, 17, 1024),
                    ctx=str(rng.choice([0, _log_int(rng, 1, 2048)])), paged=rng.random() < 0.3, tuned=rng.random() < 0.5)
    batch = rng.choice([1, 1, 2, 3, 4, 5, 6, 7, 8])
    ctx = ",".join(str(_log_int(rng, 1, 4000)) for _ in range(batch))
    return dict(kind=kind, shape=shape, layers=layers, k=rng.randint(1, 8), ctx=ctx, paged=rng.random() < 0.3,
                tuned=rng.random() < 0.5)


# -------------------------------------------------------------------------------------------- the inputs

def _gen(seed, *where):
    words = np.random.SeedSequence([int(seed) & 0x7FFFFFFF, *where]).generate_state(2)
    return torch.Generator(device=DEV).manual_seed(int(words[0]) * (1 << 31) + int(words[1]) // 2)


def _normal(seed, where, shape, std=1.0):
    return torch.randn(shape, generator=_gen(seed, *where), device=DEV, dtype=torch.float32).mul_(std).to(torch.bfloat16)


def _shape(case):
    return SHAPES[case["shape"]].with_layers(case["layers"]) if "shape" in case else HEAD_ONLY


def _layer(shape, seed, l):
    d, f, hd, hkv = shape.d_model, shape.ffn, shape.n_heads * shape.head_dim, shape.kv_heads * shape.head_dim
    w = {n: _normal(seed, (1, l, i), s, 0.02) for i, (n, s) in enumerate(
        [("wq", (hd, d)), ("wk", (hkv, d)), ("wv", (hkv, d)), ("wo", (d, hd)), ("w_gate", (f, d)), ("w_up", (f, d)), ("w_down", (d, f))])}
    for i, n in enumerate(("attn_norm", "ffn_norm")):  # near one, as trained norms are
        w[n] = (1 + 0.1 * _normal(seed, (2, l, i), (d,)).float()).to(torch.bfloat16)
    return w


def _head(shape, seed):
    return {"embed": _normal(seed, (3, 0), (shape.vocab + 1, shape.d_model), 0.02),
            "lm_head": _normal(seed, (3, 1), (shape.vocab, shape.d_model), 0.02),
            "final_norm": (1 + 0.1 * _normal(seed, (3, 2), (shape.d_model,)).float()).to(torch.bfloat16)}


def _model(shape, seed, batch, rows, ctx):
    # models that were dropped before are in a cycle with their layouts; the library allocates beside torch
    gc.collect()
    torch.cuda.empty_cache()
    m = binding.Model(shape, dict(_head(shape, seed), layers=[None] * shape.n_layers), max_batch=batch, max_rows=rows, max_ctx=ctx)
    for l in range(shape.n_layers):  # one layer's tensors at a time
        m.load_layer(l, _layer(shape, seed, l))
    return m


def _ctx(case):
    return [int(c) for c in case["ctx"].split(",")]


def _spec(case):
    return layout.prefill_layout(case["rows"]) if case["kind"] == "prefill" else layout.paper_layout(case["k"])


def _tokens(case, shape, seed, batch, spec):
    t = torch.randint(0, shape.vocab, (batch, spec.n_rows), generator=_gen(seed, 4), device=DEV, dtype=torch.int32)
    t[:, torch.from_numpy(spec.is_mask.astype(bool)).to(DEV)] = shape.mask_id
    return t


def _cached(case, shape, seed, l, b):
    """Keys and values of one layer and sequence, bf16 [heads, positions, head_dim]."""
    size = (shape.kv_heads, _ctx(case)[b], shape.head_dim)
    return _normal(seed, (5, l, b), size), _normal(seed, (6, l, b), size)


def _runs(v):
    """Values [heads, positions, head_dim] as the cache keeps them: runs of 32 positions, transposed."""
    pad = -v.shape[1] % 32
    v = torch.cat([v, v.new_zeros(v.shape[0], pad, v.shape[2])], 1) if pad else v
    return v.view(v.shape[0], -1, 32, v.shape[2]).transpose(2, 3)


def _capacity(case, spec):
    return -(-(max(_ctx(case)) + spec.n_groups) // 32) * 32


def _cache(case, m, shape, seed, spec):
    """The filled cache, and the parts of it that a pass writes: for every sequence the 32-position runs of keys
    and values that hold the block's positions."""
    ctx, cap = _ctx(case), _capacity(case, spec)
    batch, per = len(ctx), cap // 32
    written = [range(c // 32, (c + spec.n_groups - 1) // 32 + 1) for c in ctx]
    if case["paged"]:
        order = torch.randperm(batch * per, generator=_gen(seed, 7), device=DEV).to(torch.int32)
        kv = binding.PagedKV(binding.PagePool(m, batch * per), order.view(batch, per).contiguous(), torch.tensor(ctx, dtype=torch.int32, device=DEV))
        kk, vv = kv.pool.k_view(), kv.pool.v_view()
        page = kv.table.long()
        for l in range(shape.n_layers):
            for b, c in enumerate(ctx):
                k, v = _cached(case, shape, seed, l, b)
                if c:
                    at = page[b, : -(-c // 32)]
                    kk[l, at] = _runs(k).transpose(2, 3).transpose(0, 1)
                    vv[l, at] = _runs(v).transpose(0, 1)
        page = page.cpu().tolist()
        out = {"k": [kk[:, page[b][r]] for b in range(batch) for r in written[b]],
               "v": [vv[:, page[b][r]] for b in range(batch) for r in written[b]]}
    else:
        kv = m.kv_cache(batch, cap)
        kk, vv = kv.k_view(), kv.v_view()
        for l in range(shape.n_layers):
            for b, c in enumerate(ctx):
                k, v = _cached(case, shape, seed, l, b)
                kk[l, b, :, :c] = k
                vv[l, b, :, : -(-c // 32)] = _runs(v)
        kv.len.copy_(torch.tensor(ctx, dtype=torch.int32))
        out = {"k": [kk[:, b, :, r[0] * 32:(r[-1] + 1) * 32] for b, r in enumerate(written)],
               "v": [vv[:, b, :, r[0]:r[-1] + 1] for b, r in enumerate(written)]}
    kv.set_len_bound(max(ctx))
    return kv, out


@dataclass
class State:
    call: object
    out: object


def prepare(case, seed):
    if case["kind"] == "loss":
        return _prepare_loss(case, seed)
    if case["kind"] == "sample":
        return _prepare_sample(case, seed)
    shape, spec, batch = _shape(case), _spec(case), len(_ctx(case))
    m = _model(shape, seed, batch, spec.n_rows, _capacity(case, spec))
    kv, written = _cache(case, m, shape, seed, spec)
    lay = m.layout(spec)
    tokens = _tokens(case, shape, seed, batch, spec)
    if case["tuned"]:
        m.tune_rows(batch * spec.n_rows)  # once per model and row count, as the decoder and the batcher do
    if case["kind"] == "prefill":
        return State(lambda: m.prefill(tokens, lay, kv), written)
    out = binding.StepOut(m, batch, spec.n_rows, case["k"], next_rows=spec.n_rows)
    # every row's logits and what the verification made of them; the rows' argmax and the drawn tokens are
    # functions of the logits that a last-bit tie can change, the accepted count is what the commit takes
    res = dict(written, logits=out.logits, accepted=out.accepted_len)
    return State(lambda: m.step(tokens, lay, kv, out, next_layout=lay), res)


def _sample_inputs(case, seed):
    """Logits with a few likely tokens in every row, candidates that often are one of them."""
    spec, B, V, K = layout.paper_layout(case["k"]), case["batch"], HEAD_ONLY.vocab, case["top_k"]
    g = _gen(seed, 8)
    L, G, C = spec.n_rows, spec.n_groups, case["k"]
    rnd = lambda *s: torch.rand(s, generator=g, device=DEV)  # noqa: E731
    logits = torch.randn((B, L, V), generator=g, device=DEV).mul_(2.0)
    likely = torch.randint(0, V, (B, L, 16), generator=g, device=DEV)
    logits.scatter_add_(2, likely, 6.0 + 4.0 * rnd(B, L, 16))
    tokens = torch.full((B, L), HEAD_ONLY.mask_id, dtype=torch.int32, device=DEV)
    real = torch.from_numpy(np.flatnonzero(spec.is_mask == 0)).to(DEV)
    tokens[:, real[0]] = torch.randint(0, V, (B,), generator=g, device=DEV).int()
    tokens[:, real[1:]] = logits[:, real[:-1]].argmax(2).int()
    p_c = 0.2 + 0.8 * rnd(B, C)
    uniforms = rnd(B, G + C)
    draft_ids = likely[:, :C, :1].repeat(1, 1, K).int()
    draft_ids[:, :, 1:] = torch.randint(0, V, (B, C, K - 1), generator=g, device=DEV).int()
    draft_probs = torch.softmax(4.0 * rnd(B, C, K), 2)
    return spec, logits, tokens, p_c, uniforms, draft_ids, draft_probs


def _prepare_sample(case, seed):
    spec, logits, tokens, p_c, uniforms, ids, probs = _sample_inputs(case, seed)
    B, k, K = case["batch"], case["k"], case["top_k"]
    m = _model(HEAD_ONLY, seed, B, spec.n_rows, 64)
    lay = m.layout(spec)
    out = binding.SampleOut(m, B, spec.n_groups, k, K, next_rows=spec.n_rows)
    kw = dict(top_k=K, top_p=case["top_p"], residual=case["residual"], next_layout=lay)
    if case["residual"]:
        kw.update(draft_ids=ids, draft_probs=probs)
    res = {n: getattr(out, n) for n in ("accepted_len", "extra", "new_cands", "new_pc", "new_ids", "new_probs", "next_tokens", "ratios")}
    return State(lambda: m.sample_verify(logits, tokens, lay, p_c, uniforms, out, **kw), res)


def _loss_inputs(case, seed):
    rows, V = case["rows"], case["vocab"]
    g = _gen(seed, 9)
    logits = torch.randn((rows, V), generator=g, device=DEV).mul_(2.0)
    labels = torch.randint(0, V, (rows,), generator=g, device=DEV, dtype=torch.int32)
    labels[: rows // 3] = -1  # the prompt
    return logits, labels


def _prepare_loss(case, seed):
    logits, labels = _loss_inputs(case, seed)
    shape = HEAD_ONLY if case["vocab"] == HEAD_ONLY.vocab else SHAPES["tiny"].with_layers(1)
    m = _model(shape, seed, 1, 36, 64)
    row_loss = torch.empty(case["rows"], dtype=torch.float32, device=DEV)

    def call():
        return {"row_loss": row_loss, **dict(zip(("loss", "terms"), m.sar_loss(logits, labels, row_loss)))}
    return State(call, None)


def run(state):
    r = state.call()
    return r if state.out is None else state.out


# ------------------------------------------------------------------------------- what a pass cannot do without

def work(case):
    if case["kind"] == "loss":
        kept = case["rows"] - case["rows"] // 3
        return {"bytes": 4.0 * kept * case["vocab"] + 8.0 * case["rows"], "flops": 3.0 * kept * case["vocab"]}
    if case["kind"] == "sample":
        rows = case["batch"] * (case["k"] + 1) ** 2
        # the rows the walk never reaches are not known before the first are verified: every row is read
        return {"bytes": 4.0 * rows * HEAD_ONLY.vocab + 8.0 * case["batch"] * case["k"] * case["top_k"], "flops": 0.0}
    shape, spec, ctx = _shape(case), _spec(case), _ctx(case)
    d, f, hd, hkv, N = shape.d_model, shape.ffn, shape.n_heads * shape.head_dim, shape.kv_heads * shape.head_dim, shape.n_layers
    M = len(ctx) * spec.n_rows
    qkv, rest = d * (hd + 2 * hkv), d * hd + 3 * d * f
    # a prompt chunk needs no more of its last layer than the keys and values
    full = N if case["kind"] == "step" else N - 1
    last = 0 if case["kind"] == "step" else 2 * d * hkv
    weights = full * (qkv + rest) + last
    seen = sum(spec.n_rows * c for c in ctx) + len(ctx) * spec.n_groups * spec.n_rows / 2
    flops = 2.0 * M * weights + 4.0 * full * seen * hd
    moved = 2.0 * weights + 4.0 * full * hkv * sum(ctx) + 4.0 * N * hkv * spec.n_groups * len(ctx) + 2.0 * M * d
    if case["kind"] == "step":
        flops += 2.0 * M * d * shape.vocab
        moved += 2.0 * d * shape.vocab + 4.0 * M * shape.vocab
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    if case["kind"] == "loss":
        return {"rel": 1e-6, "max": 4e-6}  # float32 sums of one row
    if case["kind"] == "sample":
        return {"rel": 4e-6, "max": 4e-5}  # probabilities of at most 64 tokens in float32; ids do not differ
    # Activations carry 16 bits and sums 32; keys and values are stored as bf16, and one that lies on a
    # rounding boundary moves by a whole bf16 step when a sum in front of it changes in its last bit.
    # Measured between tilings of the same path (sums in other orders): 0.9e-4 .. 2.5e-4 on steps, up to
    # 8.3e-4 on the last keys of a prompt chunk, at most one bf16 step (0.8e-2) on a single value.
    return {"rel": 3.3e-3 if case["kind"] == "prefill" else 1e-3, "max": 3e-2}


# --------------------------------------------------------------------------------- the same in 64 bits

def exact(case, seed):
    with torch.no_grad():
        if case["kind"] == "loss":
            return _exact_loss(case, seed)
        if case["kind"] == "sample":
            return _exact_sample(case, seed)
        return _exact_forward(case, seed)


def _exact_loss(case, seed):
    logits, labels = _loss_inputs(case, seed)
    keep = labels >= 0
    terms = torch.zeros(case["rows"], dtype=torch.float64, device=DEV)
    for lo in range(0, case["rows"], 256):
        x, y = logits[lo:lo + 256].double(), labels[lo:lo + 256].long().clamp(min=0)
        terms[lo:lo + 256] = torch.logsumexp(x, 1) - x.gather(1, y[:, None])[:, 0]
    terms = torch.where(keep, terms, torch.zeros_like(terms))
    return {"row_loss": terms, "loss": terms.sum().view(1), "terms": None}


def _exact_sample(case, seed):
    """Lines 6-22 of Algorithm 1 on the lists of kept tokens, in float64; the ids come with the probabilities."""
    spec, logits, tokens, p_c, uniforms, d_ids, d_probs = _sample_inputs(case, seed)
    B, k, K, G = case["batch"], case["k"], case["top_k"], spec.n_groups
    top, ids = logits.double().topk(K, 2)
    p = torch.softmax(top, 2)
    before = p.cumsum(2) - p
    p = torch.where(before < float(np.float32(case["top_p"])), p, torch.zeros_like(p))
    p = (p / p.sum(2, keepdim=True)).cpu().numpy()
    ids, tokens, p_c, u = ids.cpu().numpy(), tokens.cpu().numpy(), p_c.double().cpu().numpy(), uniforms.double().cpu().numpy()
    real = np.flatnonzero(spec.is_mask == 0)
    new_pc, new_probs, ratios = np.zeros((B, k)), np.zeros((B, k, K)), np.full((B, max(G - 1, 1)), -1.0)
    for b in range(B):
        acc = 0
        while acc < G - 1:
            row, c = real[acc], tokens[b, real[acc + 1]]
            ratios[b, acc] = p[b, row][ids[b, row] == c].sum() / p_c[b, acc]
            if u[b, acc] > ratios[b, acc]:
                break
            acc += 1
        for j in range(k):
            q = p[b, real[acc] + 1 + j]
            at = min(int(np.searchsorted(q.cumsum(), u[b, G + j], side="right")), int((q > 0).sum()) - 1)
            new_pc[b, j], new_probs[b, j] = q[at], q
    return {"accepted_len": None, "extra": None, "new_cands": None, "new_pc": torch.from_numpy(new_pc), "new_ids": None,
            "new_probs": torch.from_numpy(new_probs), "next_tokens": None, "ratios": torch.from_numpy(ratios)}


def _exact_forward(case, seed):
    """The decoder of the step or the chunk, float64 throughout (the block's own keys and values included)."""
    shape, spec, ctx = _shape(case), _spec(case), _ctx(case)
    B, L, G, dh, H, Hkv = len(ctx), spec.n_rows, spec.n_groups, shape.head_dim, shape.n_heads, shape.kv_heads
    f64 = torch.float64
    mask, group = spec.is_mask.astype(bool), spec.group
    # a token is visible to every later row, a mask to later masks of its own group
    idx = np.arange(L)
    vis = (idx[None, :] <= idx[:, None]) & (~mask[None, :] | (mask[:, None] & (group[None, :] == group[:, None])))
    rel = torch.from_numpy(vis.sum(1) - 1).to(DEV)
    vis = torch.from_numpy(vis).to(DEV)
    real = torch.from_numpy(np.flatnonzero(~mask)).to(DEV)
    head = _head(shape, seed)
    x = head["embed"][_tokens(case, shape, seed, B, spec).long()].to(f64)
    freq = float(np.float32(shape.rope_base)) ** (-torch.arange(0, dh, 2, dtype=f64, device=DEV) / dh)

    def mul(v, w):
        return v @ w.to(f64).t()

    def norm(v, w):
        return v * torch.rsqrt((v * v).mean(-1, keepdim=True) + float(np.float32(shape.rms_eps))) * w.to(f64)

    def rotate(v, pos):  # [L, heads, dh]
        a = pos.to(f64)[:, None, None] * freq
        lo, hi = v[..., : dh // 2], v[..., dh // 2:]
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)

    new_k, new_v = [[None] * shape.n_layers for _ in ctx], [[None] * shape.n_layers for _ in ctx]
    for l in range(shape.n_layers):
        w = _layer(shape, seed, l)
        h = norm(x, w["attn_norm"])
        q, k, v = (mul(h, w[n]).view(B, L, -1, dh) for n in ("wq", "wk", "wv"))
        att = torch.empty(B, L, H * dh, dtype=f64, device=DEV)
        last = case["kind"] == "prefill" and l == shape.n_layers - 1
        for b, c in enumerate(ctx):
            pos = c + rel
            qb, kb, vb = rotate(q[b], pos).transpose(0, 1), rotate(k[b], pos).transpose(0, 1).contiguous(), v[b].transpose(0, 1).contiguous()
            ck, cv = _cached(case, shape, seed, l, b)
            r0 = c // 32 * 32
            new_k[b][l] = torch.cat([ck[:, r0:].to(f64), kb[:, real]], 1)
            new_v[b][l] = torch.cat([cv[:, r0:].to(f64), vb[:, real]], 1)
            if last:
                continue
            for h0 in range(H):
                g = h0 // (H // Hkv)
                kk, vv = torch.cat([ck[g].to(f64), kb[g]]), torch.cat([cv[g].to(f64), vb[g]])
                s = qb[h0] @ kk.t() / math.sqrt(dh)
                s[:, c:].masked_fill_(~vis, -math.inf)
                att[b, :, h0 * dh:(h0 + 1) * dh] = torch.softmax(s, 1) @ vv
        if last:
            break
        x = x + mul(att, w["wo"])
        h = norm(x, w["ffn_norm"])
        x = x + mul(torch.nn.functional.silu(mul(h, w["w_gate"])) * mul(h, w["w_up"]), w["w_down"])

    out = {"k": [], "v": []}
    for b in range(B):
        kb, vb = torch.stack(new_k[b]), torch.stack(new_v[b])  # layers, heads, positions from the first written run on
        kr = torch.stack([_runs(t).transpose(2, 3) for t in kb])  # layers, heads, runs, 32, dh
        vr = torch.stack([_runs(t) for t in vb])
        if case["paged"]:
            out["k"] += [kr[:, :, r] for r in range(kr.shape[2])]
            out["v"] += [vr[:, :, r] for r in range(vr.shape[2])]
        else:
            out["k"].append(kr.flatten(2, 3))
            out["v"].append(vr)
    if case["kind"] == "step":
        out.update(logits=mul(norm(x, head["final_norm"]), head["lm_head"]), accepted=None)
    return out

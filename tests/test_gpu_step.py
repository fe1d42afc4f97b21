"""GPU parity of the auto-correct step against the CPU oracle, through the C ABI.

The oracle runs in float64 with the one rounding the implementation's storage format imposes
(k after rotary and v are cached in bf16).  Bar: logits within 2e-2 absolute (in practice within
2e-3: activations feed the matrix units as split bf16 hi + lo planes); token ids, accepted
lengths and new candidates identical except where the oracle's top-2 logits are closer than
1e-3; cache rows identical except for values that sit on a bf16 rounding boundary.
"""
import numpy as np
import pytest

from oracle import space_oracle as so
from space_inputs import SHAPES, all_weights, prompt_tokens
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    return gc.require_gpu()


def _setup(shape_name, max_batch=1, max_rows=64, seed=0, attn=None):
    shape = SHAPES[shape_name]
    w = all_weights(shape, seed=seed)
    gm = gc.make_gpu_model(shape, w, max_batch=max_batch, max_rows=max_rows, attn=attn)
    om = gc.oracle_model(shape, w)
    return shape, gm, om


def _run_step(torch, gm, cache, spec, tokens_np, next_spec=None, batch=1):
    from paper_2402_11809_amd import binding
    lay = gm.layout(spec)
    nxt = gm.layout(next_spec) if next_spec is not None else None
    max_c = max(1, int(spec.is_mask.sum()))
    out = binding.StepOut(gm, batch, spec.n_rows, max_c, next_rows=next_spec.n_rows if next_spec else 0)
    t = torch.from_numpy(np.ascontiguousarray(tokens_np, dtype=np.int32)).cuda()
    gm.step(t, lay, cache, out, next_layout=nxt)
    torch.cuda.synchronize()
    assert gm.device_faults() == 0
    return out


@pytest.mark.parametrize("shape_name,k,attn", [("tiny", 1, None), ("tiny", 3, None), ("tiny", 4, None),
                                               ("tiny", 5, None), ("small128", 2, None), ("small128", 5, None),
                                               ("small128", 6, None), ("tiny", 3, "split"), ("small128", 5, "split"),
                                               ("tiny", 1, "split"), ("gqa-small", 3, None), ("gqa-small", 5, "split"),
                                               ("gqa128", 5, None), ("gqa128", 6, None)])
def test_step_matches_oracle(torch_mod, shape_name, k, attn):
    """One step after a real prefill: logits, ids, verification outputs, staged and committed K/V.
    Blocks of at most 48 rows run the one-workgroup-per-head attention kernel unless attn says
    otherwise; k = 6 (49 rows) and the 16-row prefill chunks of the "split" cases run the other one.
    The gqa shapes have fewer key/value heads than query heads (grouped-query attention)."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup(shape_name, max_rows=64, attn=attn)
    n_prompt = 45
    prompt = prompt_tokens(shape, seed=1, n=n_prompt)
    dec = SpaceDecoder(gm, k, batch=1, capacity=128, prefill_chunk=16)
    dec.prefill(prompt[:, :-1])
    okv = so.OracleKV(om)
    so.prefill(om, okv, prompt[0, :-1])
    # committed prompt rows agree
    torch.cuda.synchronize()
    assert int(dec.kv.len.cpu()[0]) == n_prompt - 1 == okv.length
    for l in range(shape.n_layers):
        gk, gv = gc.download_kv_rows(dec.kv, l, 0, 0, n_prompt - 1)
        gc.assert_bf16_close(gk, okv.k[l], f"prefill K layer {l}", min_same=0.97 if l == 0 else 0.9)
        gc.assert_bf16_close(gv, okv.v[l], f"prefill V layer {l}", min_same=0.97 if l == 0 else 0.9)
    # candidates: the oracle's own greedy continuation with the last one corrupted
    truth = so.ar_greedy(om, prompt[0], k + 1)[n_prompt:]
    cands = list(truth[:k])
    if k >= 2:
        cands[k - 1] = (cands[k - 1] + 1) % shape.vocab
    spec = lo.paper_layout(k)
    toks, is_mask = so.extended_input([int(prompt[0, -1])], cands, k, shape.mask_id)
    assert np.array_equal(is_mask.astype(np.uint8), spec.is_mask)
    out = _run_step(torch, gm, dec.kv, spec, toks[None], next_spec=spec)
    ref, ks, vs, pos = so.space_step_cached(om, okv, int(prompt[0, -1]), cands, k, commit=False)
    g_logits = out.logits.cpu().numpy()[0].astype(np.float64)
    err = np.abs(g_logits - ref.logits).max()
    print(f"{shape_name} k={k}: max |logit diff| = {err:.3e}")
    assert err < gc.LOGIT_TIGHT < gc.LOGIT_TOL
    g_arg = out.argmax.cpu().numpy()[0]
    ties = gc.check_ids(g_arg, ref.logits, "argmax")
    if ties == 0:
        assert int(out.accepted_len.cpu()[0]) == ref.accepted == (k - 1 if k >= 2 else k)
        assert int(out.bonus.cpu()[0]) == ref.emitted[-1]
        assert list(out.new_cands.cpu().numpy()[0][:k]) == ref.new_cands
        nxt, _ = so.extended_input([ref.emitted[-1]], ref.new_cands, k, shape.mask_id)
        assert list(out.next_tokens.cpu().numpy()[0]) == list(nxt)
    # K/V of the accepted rows sit at their final slots; commit makes them visible
    a = int(out.accepted_len.cpu()[0])
    gm.kv_commit(dec.kv, out.accepted_len)
    torch.cuda.synchronize()
    assert int(dec.kv.len.cpu()[0]) == n_prompt - 1 + a + 1
    rows = [g * (k + 1) for g in range(a + 1)]
    for l in range(shape.n_layers):
        gk, gv = gc.download_kv_rows(dec.kv, l, 0, n_prompt - 1, n_prompt + a)
        gc.assert_bf16_close(gk, ks[l][rows], f"committed K layer {l}", min_same=0.97 if l == 0 else 0.9)
        gc.assert_bf16_close(gv, vs[l][rows], f"committed V layer {l}", min_same=0.97 if l == 0 else 0.9)
    # rollback takes them away again
    gm.kv_rollback(dec.kv, None, n_all=a + 1)
    torch.cuda.synchronize()
    assert int(dec.kv.len.cpu()[0]) == n_prompt - 1


@pytest.mark.parametrize("k", [3, 5])
def test_forced_acceptance_lengths(torch_mod, k):
    """Every acceptance length 0..k (closed form: longest prefix equal to the greedy continuation)."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup("tiny")
    prompt = prompt_tokens(shape, seed=2, n=30)
    truth = so.ar_greedy(om, prompt[0], k + 1)[30:]
    dec = SpaceDecoder(gm, k, capacity=96, prefill_chunk=32)
    dec.prefill(prompt[:, :-1])
    spec = lo.paper_layout(k)
    for j in range(k + 1):
        cands = list(truth[:k])
        if j < k:
            cands[j] = (cands[j] + 7) % shape.vocab
        toks, _ = so.extended_input([int(prompt[0, -1])], cands, k, shape.mask_id)
        out = _run_step(torch, gm, dec.kv, spec, toks[None])
        assert int(out.accepted_len.cpu()[0]) == j
        assert int(out.bonus.cpu()[0]) == truth[j]
        # nothing committed: the next variant sees the same cache
        gm.kv_rollback(dec.kv, None, n_all=0)


@pytest.mark.parametrize("shape_name,k,n_new", [("tiny", 4, 32), ("tiny", 2, 24), ("small128", 5, 24),
                                                ("gqa-small", 4, 24)])
def test_generate_is_lossless(torch_mod, shape_name, k, n_new):
    """Config 1: greedy SPACE on the GPU == plain greedy AR decoding (oracle) == GPU one-token
    decoding, token for token."""
    torch = torch_mod
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup(shape_name)
    prompt = prompt_tokens(shape, seed=0, n=64)
    dec = SpaceDecoder(gm, k, capacity=256, prefill_chunk=64)
    seqs, hist = dec.generate(prompt, n_new)
    assert all(0 <= int(h[0]) <= k for h in hist) and int(hist[0][0]) == 0
    ref = so.ar_greedy(om, prompt[0], n_new)
    got = [int(t) for t in seqs[0]]
    if got != ref:
        # tolerated only at a near tie of the oracle's logits
        first = next(i for i, (a, b) in enumerate(zip(got, ref)) if a != b)
        logits = so.causal_forward(om, ref[:first])[-1]
        assert gc.top2_gap(logits) < gc.TIE_GAP, f"diverged at {first} with gap {gc.top2_gap(logits)}"
    # GPU autoregressive decoding through the same ABI (k = 0 blocks of one row)
    gm2 = gc.make_gpu_model(shape, all_weights(shape, seed=0), max_rows=64)
    dec0 = SpaceDecoder(gm2, 0, capacity=256, prefill_chunk=64)
    seq0, _ = dec0.generate(prompt, n_new)
    assert [int(t) for t in seq0[0]] == got
    print(f"{shape_name} k={k}: {n_new} tokens in {len(hist)} invocations")


def test_graph_replayed_loop_equals_the_host_driven_loop(torch_mod):
    """Algorithm 1's while loop as the product runs it: one iteration (step + commit) captured into a HIP
    graph and replayed, the host looking at the counters only after as many replays as the missing tokens
    need at least.  It must emit what the kernel-by-kernel loop emits, invocation by invocation, which in
    turn is the oracle's greedy sequence; a decoder can be used again; a batch works the same way."""
    torch = torch_mod
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup("small128", max_batch=3)
    k, n_new = 3, 30
    prompt = prompt_tokens(shape, seed=5, n=48, batch=3)
    outs = []
    for graph in (True, False):
        dec = SpaceDecoder(gm, k, batch=3, capacity=256, prefill_chunk=32, graph=graph)
        seqs, hist = dec.generate(prompt, n_new)
        outs.append((seqs.copy(), [h.copy() for h in hist], dec.iterations, dec.kv.len.cpu().numpy().copy()))
        if graph:  # again on the same decoder (and its captured graphs are dropped with the old state)
            seqs2, hist2 = dec.generate(prompt, n_new)
            assert np.array_equal(seqs, seqs2) and len(hist) == len(hist2)
            assert all(np.array_equal(a, b) for a, b in zip(hist, hist2))
    (sa, ha, ia, la), (sb, hb, ib, lb) = outs
    assert np.array_equal(sa, sb) and ia == ib == len(ha) == len(hb)
    assert all(np.array_equal(a, b) for a, b in zip(ha, hb)) and np.array_equal(la, lb)
    assert np.array_equal(la, 47 + np.sum([h + 1 for h in ha], axis=0))
    # no invocation ran that was not needed: before the last one some sequence was still short
    short = np.sum([h + 1 for h in ha[:-1]], axis=0)
    assert (short < n_new).any()
    for b in range(3):
        ref = so.ar_greedy(om, prompt[b], n_new)
        got = [int(t) for t in sa[b]]
        if got != ref:
            first = next(i for i, (x, y) in enumerate(zip(got, ref)) if x != y)
            assert gc.top2_gap(so.causal_forward(om, ref[:first])[-1]) < gc.TIE_GAP
    assert gm.device_faults() == 0


def test_eos_stops_the_sequence(torch_mod):
    """EOS check of Algorithm 1 on the device: the output ends in front of the first EOS token, also
    when it falls in the middle of a step's accepted run; the flag is sticky."""
    torch = torch_mod
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup("tiny")
    prompt = prompt_tokens(shape, seed=0, n=40)
    ref = so.ar_greedy(om, prompt[0], 20)
    gen = ref[40:]
    for pos in (0, 2, 9):
        eos = gen[pos]
        first = gen.index(eos)
        for k in (2, 4):
            dec = SpaceDecoder(gm, k, capacity=128, prefill_chunk=32, eos_id=eos)
            seqs, hist = dec.generate(prompt, 20)
            oracle_out, _ = so.space_generate(om, [int(t) for t in prompt[0]], k, 20, eos_id=eos)
            n = int(dec.lengths[0])
            assert n == first == len(oracle_out) - 40
            assert [int(t) for t in seqs[0][: 40 + n]] == oracle_out
            assert int(dec.out.finished.cpu()[0]) == 1
            # one more step appends nothing
            gm.step(dec.out.next_tokens, dec.lay_step, dec.kv, dec.out, next_layout=dec.lay_step)
            torch.cuda.synchronize()
            assert int(dec.out.emit_len.cpu()[0]) == n


def test_first_step_layout_and_prefill_chunking(torch_mod):
    """[x_l, M^k] alone gives the same extra token / candidates as the full block with dummies, and
    the cache does not depend on how the prompt was chunked."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup("tiny")
    k = 4
    prompt = prompt_tokens(shape, seed=3, n=41)
    d1 = SpaceDecoder(gm, k, capacity=96, prefill_chunk=7)
    d2 = SpaceDecoder(gm, k, capacity=96, prefill_chunk=40)
    d1.prefill(prompt[:, :-1])
    d2.prefill(prompt[:, :-1])
    torch.cuda.synchronize()
    k1 = d1.kv.k_view()[:, 0, :, :40].float().cpu().numpy()
    k2 = d2.kv.k_view()[:, 0, :, :40].float().cpu().numpy()
    assert np.mean(k1 == k2) > 0.995 and np.abs(k1 - k2).max() < 0.05
    first = np.array([[int(prompt[0, -1])] + [shape.mask_id] * k])
    o1 = _run_step(torch, gm, d1.kv, lo.first_step_layout(k), first)
    full, _ = so.extended_input([int(prompt[0, -1])], [0] * k, k, shape.mask_id)
    o2 = _run_step(torch, gm, d1.kv, lo.paper_layout(k), full[None])
    assert int(o1.accepted_len.cpu()[0]) == 0
    assert int(o1.bonus.cpu()[0]) == int(o2.argmax.cpu()[0, 0])
    assert list(o1.new_cands.cpu().numpy()[0]) == list(o2.argmax.cpu().numpy()[0, 1:k + 1])
    assert np.abs(o1.logits.cpu().numpy()[0] - o2.logits.cpu().numpy()[0, :k + 1]).max() < 1e-4


@pytest.mark.parametrize("shape_name,n_prompt,chunk", [("small128", 411, 410), ("small128", 411, 200), ("gqa-small", 300, 299),
                                                        ("tiny", 1001, 1000)])
def test_long_prompt_chunks_match_oracle(torch_mod, shape_name, n_prompt, chunk):
    """Prompt chunks of hundreds of rows through space_prefill (no LM head, last layer stops after its
    keys and values; projections in 96- and 128-row passes, attention over a long causal block): the
    cache they leave equals the oracle's, and so does the auto-correct step that follows."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup(shape_name, max_rows=chunk)
    k = 3
    prompt = prompt_tokens(shape, seed=5, n=n_prompt)
    dec = SpaceDecoder(gm, k, capacity=(n_prompt + 64 + 31) // 32 * 32, prefill_chunk=chunk)
    dec.prefill(prompt[:, :-1])
    torch.cuda.synchronize()
    assert gm.device_faults() == 0 and int(dec.kv.len.cpu()[0]) == n_prompt - 1
    okv = so.OracleKV(om)
    so.prefill(om, okv, prompt[0, :-1])
    n = n_prompt - 1
    for l in range(shape.n_layers):      # keys and values of every layer, bf16 on both sides
        kd = dec.kv.k_view()[l, 0, :, :n].float().cpu().numpy()                  # [Hkv, n, dh]
        ko = np.transpose(okv.k[l][:n], (1, 0, 2))
        vd = dec.kv.v_rows()[l, 0, :, :n].float().cpu().numpy()
        vo = np.transpose(okv.v[l][:n], (1, 0, 2))
        for got, want in ((kd, ko), (vd, vo)):
            # both are bf16 roundings of values that differ by the fp32 path's error (bounded like the
            # logits' tight bar): one bf16 step where they fall on different sides, plus that error
            ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(want), 2.0 ** -10))) - 7)
            assert np.all(np.abs(got - want) <= 1.001 * ulp + gc.LOGIT_TIGHT) and np.mean(got != want) < 0.15
    truth = so.ar_greedy(om, prompt[0], k)[n_prompt:]
    cands = truth[:2] + [(truth[2] + 1) % shape.vocab]
    toks, _ = so.extended_input([int(prompt[0, -1])], cands, k, shape.mask_id)
    out = _run_step(torch, gm, dec.kv, lo.paper_layout(k), toks[None])
    ref, _, _, _ = so.space_step_cached(om, okv, int(prompt[0, -1]), cands, k)
    assert np.abs(out.logits.cpu().numpy()[0] - ref.logits).max() < gc.LOGIT_TOL
    assert int(out.accepted_len.cpu()[0]) == ref.accepted == 2
    assert int(out.bonus.cpu()[0]) == ref.emitted[-1]
    # a block that long cannot be verified: space_step says so
    if chunk > 96:
        with pytest.raises(binding.SpaceError) as e:
            _run_step(torch, gm, dec.kv, lo.prefill_layout(chunk), prompt[:, :chunk])
        assert e.value.code == binding.SPACE_ESHAPE


@pytest.mark.parametrize("shape_name,rows,k,ctxs,paged", [
    ("64 heads", 256, 0, [40], False),           # heads of 64: a workgroup per CU, one too few (attn_sar_kernel)
    ("64 heads", 257, 0, [31], True),            # a fifth group of one row, and workgroups that share CUs
    ("64 heads of 128", 256, 0, [0], False),     # a lone prompt, a workgroup per CU, four full groups
    ("64 heads", 449, 0, [1023], False),         # two to a CU
    ("64 heads", 576, 23, [45], False),          # mask rows; more workgroups than fit at once
    ("gqa128", 993, 0, [1, 700], False),         # equal numbers of workgroups and CUs, two sequences
    ("64 heads of 128", 321, 0, [700], True),    # heads of 128 over pages, six groups
    ("gqa128", 257, 0, "ragged", True),          # ... dealt out and cut by length
    ("gqa-small", 193, 0, "ragged", False),      # a batch dealt out and cut by length, merged by whoever ends last
    ("gqa-small", 196, 13, "ragged", True),
    ("tiny", 321, 0, "ragged", False),
])
def test_attention_of_long_blocks(torch_mod, shape_name, rows, k, ctxs, paged):
    """Blocks that attn_rows_kernel takes (space_prefill) and one that it does not, prompts and blocks with mask rows, at the edges of the 64-row groups, 32-key
    chunks and 64-key stages: the first layer's attention output of every row against the oracle's, and the keys and values of
    the layer behind it."""
    torch = torch_mod
    import dataclasses
    from paper_2402_11809_amd import binding, layout as lo
    if shape_name.startswith("64 heads"):
        shape = dataclasses.replace(SHAPES["gqa-small"], n_layers=2, n_heads=64, n_kv_heads=8, head_dim=128 if "128" in shape_name else 64)
    else:
        shape = dataclasses.replace(SHAPES[shape_name], n_layers=2)
    w = all_weights(shape, seed=8)
    spec = lo.paper_layout(k) if k else lo.prefill_layout(rows)
    assert spec.n_rows == rows
    if ctxs == "ragged":
        ctxs = [(151 * b) % 690 for b in range(11)] + [700]
    B, cap = len(ctxs), -(-(max(ctxs) + spec.n_groups) // 32) * 32
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=rows, max_ctx=cap)
    om = gc.oracle_model(shape, w)
    okvs = [gc.synthetic_oracle_kv(om, seed=30 + b, ctx=c, std=0.5) for b, c in enumerate(ctxs)]
    cache = gm.kv_cache(B, cap)
    for b in range(B):
        gc.upload_oracle_kv(torch, cache, b, okvs[b])
    kv = cache
    if paged:
        per = cap // 32
        order = torch.randperm(B * per, generator=torch.Generator().manual_seed(1)).view(B, per)
        kv = binding.PagedKV(binding.PagePool(gm, B * per), order.int().cuda().contiguous(), cache.len)
        kv.set_len_bound(max(ctxs))
        for b in range(B):
            at = order[b].cuda()
            kv.pool.k_view()[:, at] = cache.k_view()[:, b].unflatten(2, (per, 32)).transpose(1, 2)
            kv.pool.v_view()[:, at] = cache.v_view()[:, b].transpose(1, 2)
    rng = np.random.default_rng(11)
    toks = rng.integers(0, shape.vocab, size=(B, rows)).astype(np.int32)
    toks[:, spec.is_mask.astype(bool)] = shape.mask_id
    gm.prefill(torch.from_numpy(toks).cuda(), gm.layout(spec), kv)
    torch.cuda.synchronize()
    assert gm.device_faults() == 0
    hd = shape.n_heads * shape.head_dim
    out = gc.decode_planes(gm.debug_buffer("attn_out"), B * rows, hd).reshape(B, rows, hd)
    if paged:
        for b in range(B):
            at = order[b].cuda()
            cache.k_view()[:, b] = kv.pool.k_view()[:, at].transpose(1, 2).flatten(2, 3)
            cache.v_view()[:, b] = kv.pool.v_view()[:, at].transpose(1, 2)
    real = gc.real_rows(spec)
    for b, c in enumerate(ctxs):
        trace = []
        _, ks, vs, _ = so.block_forward_cached(om, okvs[b], toks[b].astype(np.int64), spec.is_mask.astype(bool), k=k or None, trace=trace)
        # 2^-17 per operand and sums in 32 bits, beside the block's own keys and values that round to the other bf16 neighbour
        # (some in ten thousand, a step of 2^-8 of one of the keys of a row)
        assert np.abs(out[b] - trace[0]["attn_out"].reshape(rows, hd)).max() < 2e-3, b
        got_k, got_v = gc.download_kv_rows(cache, 1, b, c, c + len(real))
        gc.assert_bf16_close(got_k, np.asarray(ks[1])[real], f"keys of {b}", min_same=0.9)
        gc.assert_bf16_close(got_v, np.asarray(vs[1])[real], f"values of {b}", min_same=0.9)


def _batched_step_vs_oracle(torch, shape, w, B, k, tune, tol, threads=1, ctxs=None, capacity=160):
    from paper_2402_11809_amd import binding, layout as lo
    spec = lo.paper_layout(k)
    L = spec.n_rows
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=L, tune=tune)
    om = gc.oracle_model(shape, w)
    if ctxs is None:
        ctxs = [(17 * (b + 1)) % 90 + 3 for b in range(B)]
    cache = binding.KVCache(gm, B, capacity)
    okvs = []
    for b, c in enumerate(ctxs):
        okv = gc.synthetic_oracle_kv(om, seed=20 + b, ctx=c, std=0.5)
        gc.upload_oracle_kv(torch, cache, b, okv)
        okvs.append(okv)
    rng = np.random.default_rng(9)
    toks = np.zeros((B, L), dtype=np.int32)
    cands = []
    for b in range(B):
        c = [int(t) for t in rng.integers(0, shape.vocab, size=k)]
        cands.append(c)
        toks[b], _ = so.extended_input([int(rng.integers(0, shape.vocab))], c, k, shape.mask_id)
    out = _run_step(torch, gm, cache, spec, toks, batch=B)
    worst = 0.0
    for b in range(B):
        ref, _, _, _ = so.space_step_cached(om, okvs[b], int(toks[b, 0]), cands[b], k, commit=False)
        err = np.abs(out.logits.cpu().numpy()[b] - ref.logits).max()
        worst = max(worst, err)
        assert err < tol, (b, err)
        gc.check_ids(out.argmax.cpu().numpy()[b], ref.logits, f"seq {b}")
        assert int(out.accepted_len.cpu()[b]) == ref.accepted
    return worst


@pytest.mark.parametrize("shape_name,B,k,ks", [("small128", 1, 5, 0), ("small128", 4, 5, 0), ("gqa-small", 5, 4, 0), ("gqa128", 2, 8, 0),
                                                ("tiny", 7, 3, 0), ("small128", 4, 5, 1), ("small128", 6, 5, 2), ("gqa128", 2, 8, 4),
                                                ("tiny", 7, 3, 2)])
def test_many_row_projection_kernel_on_small_blocks(torch_mod, shape_name, B, k, ks):
    """The projection kernel for many rows (activation planes shared through LDS, 128-row passes), forced
    for every row count: a single ragged tile, exactly one pass, a pass plus a few rows, odd numbers of
    contraction tiles, all three epilogues; with the number of partial sums over the contraction its cost
    model picks (ks = 0) and with 1, 2 and 4 forced (what space_tune_rows may choose between).  Every
    sequence against its own oracle step."""
    shape = SHAPES[shape_name]
    tune = "wide=1" + (f",wideks={ks}" if ks else "")
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=2), B, k, tune, gc.LOGIT_TIGHT)


@pytest.mark.parametrize("shape_name,B,k,tail", [("small128", 1, 5, "1:2"), ("small128", 6, 5, "3:5"), ("gqa128", 2, 8, "2:8"), ("gqa128", 8, 5, "1:16"),
                                                 ("gqa128", 5, 5, "8:2"), ("gqa-small", 5, 4, "32:1"), ("gqa-small", 5, 4, "5:3")])
def test_pieces_cut_over_the_contraction(torch_mod, shape_name, B, k, tail):
    """The last pieces of every XCD in several parts over the contraction, forced (SPACE_TUNE widetail=pieces:parts)
    wherever a projection has that many pieces and contraction tiles: one part more than there are pipeline rounds to share, single
    rounds, pieces of every size, all epilogues; "32:1" is malformed and ignored.  Against the oracle, and two steps
    in a row on the same context give the same bits (the arrival counts are back at zero, the order of the sums does not
    depend on who arrives last)."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES[shape_name]
    w = all_weights(shape, seed=11)
    tune = "wide=1,widetail=" + tail
    _batched_step_vs_oracle(torch, shape, w, B, k, tune, gc.LOGIT_TIGHT)
    spec = lo.paper_layout(k)
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=spec.n_rows, tune=tune)
    toks = np.random.default_rng(15).integers(0, shape.vocab, size=(B, spec.n_rows)).astype(np.int32)
    cache = gm.kv_cache(B, 160)
    got = [_run_step(torch, gm, cache, spec, toks, batch=B).logits.cpu().numpy().copy() for _ in range(3)]
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])


@pytest.mark.parametrize("shape_name,B,k", [("small128", 3, 5), ("small128", 6, 5), ("gqa128", 2, 8), ("small128", 8, 5)])
def test_two_and_three_passes_on_small_models(torch_mod, shape_name, B, k):
    """Row counts of two and three passes of the weight-streaming kernel on small models, nothing forced: 108, 162, 216 and 288
    rows, all in passes (which projections take the many-row kernel by themselves: the next test)."""
    shape = SHAPES[shape_name]
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=3), B, k, None, gc.LOGIT_TIGHT)


@pytest.mark.parametrize("B,k", [(6, 3), (2, 6), (12, 3), (13, 3), (9, 5)])
def test_projection_kernels_by_rounds_of_workgroups(torch_mod, B, k):
    """Where the many-row kernel takes over, per projection and nothing forced: 96 rows (one pass: none), 98 and 192 rows (two
    passes: gate / up in 376 short workgroups stays with them, the LM head in 258 long ones and QKV in 384 do not), 208 and
    324 rows (three and four: gate / up goes too, O and down stay until theirs exceed a workgroup per CU)."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["gqa128"], n_layers=1, n_kv_heads=8, ffn=6000, vocab=16500)
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=4), B, k, None, gc.LOGIT_TIGHT)


@pytest.mark.parametrize("shape_name,B,k,ctxs,tune", [
    ("gqa-small", 17, 5, "ragged", None), ("gqa-small", 17, 5, "uniform", "attn=0"),
    ("gqa-small", 17, 5, "one-long", "attn=1000000"), ("gqa128", 9, 8, "ragged", None), ("small128", 12, 5, "ragged", None),
    ("small128", 3, 5, "one-long", "attn=0"), ("gqa-small", 33, 3, "ragged", "attn=0")])
def test_batches_with_long_ragged_contexts(torch_mod, shape_name, B, k, ctxs, tune):
    """Batches whose contexts run to several hundred positions, with the attention kernel the library picks
    by itself (for these workgroup counts the one with a workgroup per (sequence, head) that sums, rotates
    and stores the block in its prologue: two partial sums of the projection, three items per thread) and
    with either one forced: ragged lengths, equal lengths, one long sequence among short ones, and a block of
    two query groups (rotary and store in a pass of their own); up to 33 sequences x 8 heads (more
    workgroups than CUs).  Every sequence against its own oracle step."""
    shape = SHAPES[shape_name]
    lens = {"ragged": [40 + (211 * b) % 700 for b in range(B)], "uniform": [544] * B,
            "one-long": [33 + b for b in range(B - 1)] + [760]}[ctxs]
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=5), B, k, tune, gc.LOGIT_TIGHT, ctxs=lens, capacity=800)


@pytest.mark.parametrize("B,k", [(6, 5), (2, 8), (8, 5)])
def test_measured_cut_and_split_stay_within_rounding(torch_mod, B, k):
    """space_tune_rows picks how the many-row kernel cuts the rows into workgroups (pieces of 128, 96, 64
    or 32 rows) and in how many parts the plain-sum projections add up the contraction.  The cut changes
    no bit (next test); the number of partial sums reorders fp32 additions, so whatever it picks, the
    logits stay within 1e-3 of the untuned step's (a reordered sum can move a key or value across a bf16
    rounding boundary, which shows downstream), and indices and accepted counts are the same wherever
    the untuned step's top two logits are more than 1e-3 apart.  216, 162 and 288 rows, with the many-row kernel forced (these
    projections would run in passes, which are not measured); also the call's error paths."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    shape = SHAPES["small128"]
    w = all_weights(shape, seed=4)
    spec = lo.paper_layout(k)
    L = spec.n_rows
    rng = np.random.default_rng(12)
    toks = rng.integers(0, shape.vocab, size=(B, L)).astype(np.int32)
    results = []
    for tuned, tune in ((False, "wide=1"), (True, "wide=1"), (False, "wide=0")):
        gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=L, tune=tune)
        if tuned:
            gm.tune_rows(B * L)
            gm.tune_rows(B * L)  # a second request for the same count is a no-op
            with pytest.raises(binding.SpaceError) as e:
                gm._check(gm.lib.space_tune_rows(gm.ctx, B * L + 1, None))
            assert e.value.code == binding.SPACE_ESHAPE
            with pytest.raises(binding.SpaceError) as e:
                gm._check(gm.lib.space_tune_rows(gm.ctx, 0, None))
            assert e.value.code == binding.SPACE_ESHAPE
        cache = binding.KVCache(gm, B, 160)
        om = gc.oracle_model(shape, w)
        for b in range(B):
            gc.upload_oracle_kv(torch, cache, b, gc.synthetic_oracle_kv(om, seed=40 + b, ctx=11 * b + 5, std=0.5))
        out = _run_step(torch, gm, cache, spec, toks, batch=B)
        results.append((out.logits.cpu().numpy().copy(), out.argmax.cpu().numpy().copy(), out.accepted_len.cpu().numpy().copy()))
    (l0, a0, n0), (l1, a1, n1), (passes, _, _) = results
    assert not np.array_equal(l0, passes)  # (another order of sums: what was measured is the many-row kernel)
    assert np.abs(l0 - l1).max() < 1e-3
    top2 = np.sort(l0, axis=-1)[..., -2:]
    clear = (top2[..., 1] - top2[..., 0]) > 1e-3
    assert np.array_equal(a0[clear], a1[clear])
    if clear.all():
        assert np.array_equal(n0, n1)


def test_every_row_cut_gives_the_same_bits(torch_mod):
    """288 rows = 9 groups of 32 rows, cut in every piece size and all launch orders (forced through SPACE_TUNE widecut=,
    and the many-row kernel through wide=): logits, indices and accepted counts equal the default cut's bit for bit."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    shape = SHAPES["small128"]
    w = all_weights(shape, seed=5)
    B, k = 8, 5
    spec = lo.paper_layout(k)
    L = spec.n_rows
    toks = np.random.default_rng(13).integers(0, shape.vocab, size=(B, L)).astype(np.int32)
    om = gc.oracle_model(shape, w)
    okvs = [gc.synthetic_oracle_kv(om, seed=60 + b, ctx=9 * b + 4, std=0.5) for b in range(B)]
    ref = None
    for cut in (None, "2:0:0:1:0", "0:3:0:0:0", "0:3:0:0:1", "0:1:3:0:1", "0:0:4:1:0", "1:0:2:1:1", "0:0:0:9:1", "1:1:1:0:0",
                "2:0:0:1:2", "0:1:3:0:2", "1:1:1:0:2"):
        gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=L, tune="wide=1" if cut is None else "wide=1,widecut=" + cut)
        cache = binding.KVCache(gm, B, 160)
        for b in range(B):
            gc.upload_oracle_kv(torch, cache, b, okvs[b])
        out = _run_step(torch, gm, cache, spec, toks, batch=B)
        got = (out.logits.cpu().numpy().copy(), out.argmax.cpu().numpy().copy(), out.accepted_len.cpu().numpy().copy())
        if ref is None:
            ref = got
        else:
            for x, y in zip(ref, got):
                assert np.array_equal(x, y), cut


@pytest.mark.parametrize("shape_name,B,k,ctxs", [("small128", 1, 5, [300]), ("small128", 3, 5, [5, 700, 33]), ("gqa-small", 2, 8, [500, 64]),
                                                 ("tiny", 1, 3, [790]), ("gqa128", 4, 2, [31, 32, 33, 650])])
def test_key_split_with_more_workgroups_than_chunks(torch_mod, shape_name, B, k, ctxs):
    """The key-split attention with several workgroups along the keys, sized for the longest sequence of
    the batch: sequences with fewer chunks than workgroups (those workgroups only leave the empty marker
    for the merge kernel), a nearly empty cache next to a long one, blocks of 36 rows (rotary fused), 81
    rows (two query groups), 16 and 9 rows.  Against the oracle's step, and three steps in a row on the
    same context give the same bits."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    shape = SHAPES[shape_name]
    w = all_weights(shape, seed=6)
    spec = lo.paper_layout(k)
    L = spec.n_rows
    om = gc.oracle_model(shape, w)
    okvs = [gc.synthetic_oracle_kv(om, seed=70 + b, ctx=c, std=0.5) for b, c in enumerate(ctxs)]
    rng = np.random.default_rng(14)
    toks = np.zeros((B, L), dtype=np.int32)
    cands = []
    for b in range(B):
        c = [int(t) for t in rng.integers(0, shape.vocab, size=k)]
        cands.append(c)
        toks[b], _ = so.extended_input([int(rng.integers(0, shape.vocab))], c, k, shape.mask_id)
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=L, tune="attn=0")
    cache = binding.KVCache(gm, B, 800)
    for b in range(B):
        gc.upload_oracle_kv(torch, cache, b, okvs[b])
    ref = None
    for rep in range(3):
        out = _run_step(torch, gm, cache, spec, toks, batch=B)
        got = (out.logits.cpu().numpy().copy(), out.argmax.cpu().numpy().copy(), out.accepted_len.cpu().numpy().copy())
        if ref is None:
            ref = got
            for b in range(B):
                o, _, _, _ = so.space_step_cached(om, okvs[b], int(toks[b, 0]), cands[b], k, commit=False)
                assert np.abs(got[0][b] - o.logits).max() < gc.LOGIT_TIGHT, b
                gc.check_ids(got[1][b], o.logits, f"seq {b}")
        else:
            for x, y in zip(ref, got):
                assert np.array_equal(x, y), rep


@pytest.mark.parametrize("shape_name", ["7b", "13b", "70b"])
def test_many_row_projection_kernel_at_full_width(torch_mod, shape_name):
    """One layer + LM head at the width of the 7B, 13B and 70B members of the family, 5 sequences x 81
    rows = 405 rows: the library picks the many-row kernel by itself (4 passes, the last of 21 rows;
    contraction splits; 2000 LM-head tiles).  Against the stated bar, not the tight one: in a one-layer
    random model of this width the attention output is ~30x the embedding, and with contexts of 3..88
    positions every key or value that rounds to the other bf16 neighbour (both sides round, from fp32
    and from fp64) shows in it.  Measured over the 13 M logits: 4.7e-3 at the 7B width, 1.1e-2 at the
    70B width (median row 2e-3, mean 5e-4), the same to three digits with either projection kernel."""
    shape = SHAPES[shape_name].with_layers(1)
    worst = _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=0, threads=8), 5, 8, None, gc.LOGIT_TOL)
    print(f"{shape_name} layer, 405 rows: max |logit diff| = {worst:.3e}")


def test_ragged_batch_matches_oracle(torch_mod):
    """Batch of sequences with different context lengths and candidates (config 5 in small):
    every sequence must match its own oracle step; explicit commit counts land in len."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    shape, gm, om = _setup("small128", max_batch=3, max_rows=36)
    k, B = 5, 3
    ctxs = [37, 100, 64]
    cache = binding.KVCache(gm, B, 160)
    okvs = []
    for b, c in enumerate(ctxs):
        okv = gc.synthetic_oracle_kv(om, seed=10 + b, ctx=c, std=0.5)
        gc.upload_oracle_kv(torch, cache, b, okv)
        okvs.append(okv)
    rng = np.random.default_rng(5)
    toks = np.zeros((B, 36), dtype=np.int32)
    cands = []
    for b in range(B):
        c = [int(t) for t in rng.integers(0, shape.vocab, size=k)]
        cands.append(c)
        toks[b], _ = so.extended_input([int(rng.integers(0, shape.vocab))], c, k, shape.mask_id)
    spec = lo.paper_layout(k)
    out = _run_step(torch, gm, cache, spec, toks, batch=B)
    for b in range(B):
        ref, ks, vs, pos = so.space_step_cached(om, okvs[b], int(toks[b, 0]), cands[b], k, commit=False)
        err = np.abs(out.logits.cpu().numpy()[b] - ref.logits).max()
        assert err < gc.LOGIT_TOL, (b, err)
        gc.check_ids(out.argmax.cpu().numpy()[b], ref.logits, f"seq {b}")
    forced = torch.tensor([0, 5, 2], dtype=torch.int32, device="cuda")
    gm.kv_commit(cache, forced)
    torch.cuda.synchronize()
    assert list(cache.len.cpu().numpy()) == [ctxs[0] + 1, ctxs[1] + 6, ctxs[2] + 3]
    ref, ks, vs, pos = so.space_step_cached(om, okvs[1], int(toks[1, 0]), cands[1], k, commit=False)
    gk, gv = gc.download_kv_rows(cache, 2, 1, ctxs[1], ctxs[1] + 6)
    gc.assert_bf16_close(gk, ks[2][[g * 6 for g in range(6)]], "forced commit K", min_same=0.9)
    gc.assert_bf16_close(gv, vs[2][[g * 6 for g in range(6)]], "forced commit V", min_same=0.9)


@pytest.mark.parametrize("attn", [None, "split"])
def test_empty_cache_and_mixed_lengths(torch_mod, attn):
    """Degenerate contexts: decoding from a one-token prompt (the first blocks run against an empty
    or nearly empty cache), and a batch in which one sequence has nothing cached while another has
    several chunks."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    from paper_2402_11809_amd.runtime import SpaceDecoder
    shape, gm, om = _setup("tiny", max_batch=2, attn=attn)
    k = 3
    prompt = prompt_tokens(shape, seed=9, n=1)
    dec = SpaceDecoder(gm, k, batch=1, capacity=64, prefill_chunk=16)
    seq, hist = dec.generate(prompt, 10)
    ref = so.ar_greedy(om, prompt[0], 10)
    got = [int(t) for t in seq[0]]
    if got != ref:
        first = next(i for i, (a, b) in enumerate(zip(got, ref)) if a != b)
        assert gc.top2_gap(so.causal_forward(om, ref[:first])[-1]) < gc.TIE_GAP
    # batch of two: sequence 0 empty, sequence 1 with 70 cached positions
    cache = binding.KVCache(gm, 2, 128)
    okv0 = so.OracleKV(om)
    okv1 = gc.synthetic_oracle_kv(om, seed=8, ctx=70, std=0.5)
    gc.upload_oracle_kv(torch, cache, 1, okv1)
    spec = lo.paper_layout(k)
    rng = np.random.default_rng(3)
    toks = np.zeros((2, spec.n_rows), dtype=np.int32)
    for b in range(2):
        toks[b], _ = so.extended_input([int(rng.integers(0, shape.vocab))], [int(t) for t in rng.integers(0, shape.vocab, size=k)],
                                       k, shape.mask_id)
    out = _run_step(torch, gm, cache, spec, toks, batch=2)
    for b, okv in enumerate((okv0, okv1)):
        ref_logits, _, _, _ = so.block_forward_cached(om, okv, toks[b], spec.is_mask.astype(bool), k)
        err = np.abs(out.logits.cpu().numpy()[b] - ref_logits).max()
        assert err < gc.LOGIT_TIGHT, (b, err)
        gc.check_ids(out.argmax.cpu().numpy()[b], ref_logits, f"sequence {b}")


def test_layers_handed_over_one_by_one(torch_mod):
    """space_load_layer: a model whose layers arrive after space_init gives bit-identical outputs; a step
    before the last layer arrived is refused."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    shape = SHAPES["tiny"]
    w = all_weights(shape, seed=0)
    gm = gc.make_gpu_model(shape, w, max_rows=16)
    dev_w = binding.weights_to_device(w)
    layers = dev_w["layers"]
    gm2 = binding.Model(shape, dict(dev_w, layers=[None] * shape.n_layers), max_batch=1, max_rows=16)
    spec = lo.paper_layout(3)
    toks = np.random.default_rng(0).integers(0, shape.vocab, size=(1, spec.n_rows)).astype(np.int32)
    toks[0, spec.is_mask == 1] = shape.mask_id
    c1, c2 = binding.KVCache(gm, 1, 64), binding.KVCache(gm2, 1, 64)
    gm2.load_layer(1, layers[1])
    with pytest.raises(binding.SpaceError) as e:
        _run_step(torch, gm2, c2, spec, toks)
    assert e.value.code == binding.SPACE_EINVAL
    gm2.load_layer(0, layers[0])
    with pytest.raises(binding.SpaceError):
        gm2.load_layer(0, layers[0])
    a = _run_step(torch, gm, c1, spec, toks)
    b = _run_step(torch, gm2, c2, spec, toks)
    assert torch.equal(a.logits, b.logits) and torch.equal(a.argmax, b.argmax)


def test_error_paths(torch_mod):
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    shape, gm, om = _setup("tiny", max_rows=25)
    with pytest.raises(binding.SpaceError) as e:
        gm.layout(lo.paper_layout(5))  # 36 rows > max_rows
    assert e.value.code == binding.SPACE_ECAPACITY
    bad = lo.BlockLayoutSpec(np.array([1, 0], dtype=np.uint8), np.array([0, 0], dtype=np.int32))
    with pytest.raises(binding.SpaceError) as e:
        gm.layout(bad)
    assert e.value.code == binding.SPACE_EINVAL
    cache = binding.KVCache(gm, 1, 32)
    cache.set_len_bound(30)
    spec = lo.paper_layout(4)
    out = binding.StepOut(gm, 1, 25, 4)
    t = torch.zeros(1, 25, dtype=torch.int32, device="cuda")
    with pytest.raises(binding.SpaceError) as e:
        gm.step(t, gm.layout(spec), cache, out)
    assert e.value.code == binding.SPACE_ECAPACITY
    with pytest.raises(binding.SpaceError) as e:
        gm.kv_commit(cache, None, accepted_all=0)  # nothing staged
    assert e.value.code == binding.SPACE_EINVAL
    # the verification assembles next blocks of at most 96 rows: a longer next_layout is refused on the host
    gm_long = gc.make_gpu_model(shape, all_weights(shape, seed=0), max_batch=1, max_rows=128)
    c_long = binding.KVCache(gm_long, 1, 256)
    out_long = binding.StepOut(gm_long, 1, 25, 4, next_rows=112)
    with pytest.raises(binding.SpaceError) as e:
        gm_long.step(t, gm_long.layout(spec), c_long, out_long, next_layout=gm_long.layout(lo.prefill_layout(112)))
    assert e.value.code == binding.SPACE_ESHAPE
    # an out-of-range token id is clamped and counted, not a fault of the GPU
    cache.set_len_bound(0)
    t[0, 0] = shape.vocab + 5
    gm.step(t, gm.layout(spec), cache, out)
    assert gm.device_faults() == 1
    assert gm.device_faults() == 0
    # space_prefill: same capacity checks as the step; more sequences than the scratch was sized for
    cache.set_len_bound(30)
    with pytest.raises(binding.SpaceError) as e:
        gm.prefill(t, gm.layout(spec), cache)
    assert e.value.code == binding.SPACE_ECAPACITY
    gm1 = gc.make_gpu_model(shape, all_weights(shape, seed=0), max_batch=2, max_rows=16)
    two = binding.KVCache(gm1, 2, 64)
    lay25 = lo.prefill_layout(16)
    gm1.prefill(torch.zeros(2, 16, dtype=torch.int32, device="cuda"), gm1.layout(lay25), two)   # 32 rows: fits
    gm1.kv_commit(two, None, accepted_all=15)
    assert two.len.cpu().tolist() == [16, 16]
    # a paged view with more pages per sequence than the context allows
    pool = binding.PagePool(gm1, 8)
    with pytest.raises(binding.SpaceError) as e:
        big = binding.PagedKV(pool, torch.zeros(1, 200, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
        gm1.prefill(torch.zeros(1, 16, dtype=torch.int32, device="cuda"), gm1.layout(lay25), big)
    assert e.value.code == binding.SPACE_ECAPACITY


@pytest.mark.parametrize("groups,masks,attn,shape_name", [
    (2, 1, None, "7b"), (2, 3, None, "7b"), (4, 3, None, "7b"), (4, 7, None, "7b"), (6, 5, None, "7b"),
    (2, 1, "head", "7b"), (6, 5, "head", "7b"), (6, 5, None, "70b"), (6, 5, "head", "70b"), (6, 5, None, "13b")])
def test_single_7b_layer_long_cache(torch_mod, groups, masks, attn, shape_name):
    """Config 3: one LLaMA-7B-shaped layer, block of L = groups * (1 + masks) rows under the
    semi-autoregressive mask against a cache of 4096 positions of N(0, 1) K/V.  Also at the 13B
    width and at the 70B width (grouped-query attention, 64 query heads over 8 key/value heads)."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    shape = SHAPES[shape_name].with_layers(1)
    w = all_weights(shape, seed=0, threads=8)
    gm = gc.make_gpu_model(shape, w, max_batch=1, max_rows=36, max_ctx=4224, attn=attn)
    om = gc.oracle_model(shape, w)
    ctx = 4096
    okv = gc.synthetic_oracle_kv(om, seed=3, ctx=ctx, std=1.0)
    cache = binding.KVCache(gm, 1, 4224)
    gc.upload_oracle_kv(torch, cache, 0, okv)
    spec = lo.grouped_layout(groups, masks)
    rng = np.random.default_rng(groups * 10 + masks)
    toks = rng.integers(0, shape.vocab, size=spec.n_rows).astype(np.int32)
    toks[spec.is_mask == 1] = shape.mask_id
    out = _run_step(torch, gm, cache, spec, toks[None])
    ref_logits, ks, vs, pos = so.block_forward_cached(om, okv, toks, spec.is_mask.astype(bool))
    assert list(pos) == [ctx + int(p) for p in gc.rel_pos(spec)]
    err = np.abs(out.logits.cpu().numpy()[0] - ref_logits).max()
    print(f"{shape_name} layer, L={spec.n_rows} ({groups}x(1+{masks})), ctx 4096: max |logit diff| = {err:.3e}")
    assert err < gc.LOGIT_TIGHT
    gc.check_ids(out.argmax.cpu().numpy()[0], ref_logits, "argmax")
    # greedy verification on these rows, closed form
    am = np.argmax(ref_logits, axis=-1)
    real = gc.real_rows(spec)
    acc = 0
    while acc < groups - 1 and toks[real[acc + 1]] == am[real[acc]]:
        acc += 1
    assert int(out.accepted_len.cpu()[0]) == acc
    assert int(out.bonus.cpu()[0]) == am[real[acc]]


@pytest.mark.parametrize("k,attn", [(3, None), (8, None), (3, "split"), (5, "head")])
def test_ragged_batch_of_eight_with_forced_commits(torch_mod, k, attn):
    """Config 5 in small: 8 sequences, ragged context lengths, blocks of (k+1)^2 rows (up to 648 rows in
    total, i.e. several projection passes), accepted lengths drawn from a geometric law and passed to
    the commit explicitly; afterwards len and the committed rows are checked."""
    torch = torch_mod
    from paper_2402_11809_amd import binding, layout as lo
    from space_inputs import geometric_accept_lengths, ragged_context_lengths
    L = (k + 1) ** 2
    shape, gm, om = _setup("small128", max_batch=8, max_rows=L, attn=attn)
    B = 8
    ctxs = [int(c) for c in ragged_context_lengths(seed=4, batch=B, lo=16, hi=300)]
    cache = binding.KVCache(gm, B, 352)
    okvs = []
    for b, c in enumerate(ctxs):
        okv = gc.synthetic_oracle_kv(om, seed=20 + b, ctx=c, std=0.5)
        gc.upload_oracle_kv(torch, cache, b, okv)
        okvs.append(okv)
    rng = np.random.default_rng(k)
    toks = np.zeros((B, L), dtype=np.int32)
    cands = []
    for b in range(B):
        c = [int(t) for t in rng.integers(0, shape.vocab, size=k)]
        cands.append(c)
        toks[b], _ = so.extended_input([int(rng.integers(0, shape.vocab))], c, k, shape.mask_id)
    out = _run_step(torch, gm, cache, lo.paper_layout(k), toks, batch=B)
    refs = []
    for b in range(B):
        ref, ks, vs, pos = so.space_step_cached(om, okvs[b], int(toks[b, 0]), cands[b], k, commit=False)
        refs.append((ref, ks, vs))
        err = np.abs(out.logits.cpu().numpy()[b] - ref.logits).max()
        assert err < gc.LOGIT_TIGHT, (b, err)
        ties = gc.check_ids(out.argmax.cpu().numpy()[b], ref.logits, f"seq {b}")
        if ties == 0:
            assert int(out.accepted_len.cpu()[b]) == ref.accepted
    forced_np = geometric_accept_lengths(seed=4, batch=B, k=k)
    assert forced_np.min() >= 0 and forced_np.max() <= k
    forced = torch.from_numpy(forced_np).cuda()
    gm.kv_commit(cache, forced)
    torch.cuda.synchronize()
    assert list(cache.len.cpu().numpy()) == [c + int(a) + 1 for c, a in zip(ctxs, forced_np)]
    for b in (0, B - 1):
        a = int(forced_np[b])
        rows = [g * (k + 1) for g in range(a + 1)]
        gk, gv = gc.download_kv_rows(cache, 1, b, ctxs[b], ctxs[b] + a + 1)
        gc.assert_bf16_close(gk, refs[b][1][1][rows], f"seq {b} K", min_same=0.9)
        gc.assert_bf16_close(gv, refs[b][2][1][rows], f"seq {b} V", min_same=0.9)
    # a per-sequence rollback undoes the commit
    gm.kv_rollback(cache, forced + 1)
    torch.cuda.synchronize()
    assert list(cache.len.cpu().numpy()) == ctxs


@pytest.mark.parametrize("shape_name,B,k,tune", [
    ("tiny", 1, 1, None),                                        # 4 rows: what the library picks by itself
    ("tiny", 2, 4, "resid=48"),                                  # 50 rows: two more than the kernel takes
    ("tiny", 3, 3, "resid=48"),                                  # 48 rows, three full row tiles
    ("small128", 1, 5, "resid=48"),                              # a ragged third tile
    ("small128", 2, 3, "resid=48,qkv=2:1,o=2:3,gu=4:1,dn=2:1"),  # packings with 12 and with 4 contraction ranges
    ("gqa128", 1, 2, "resid=48,o=8:8,dn=6:2"),                   # more contraction ranges than tiles, 9 rows
    ("wide-residual", 1, 2, "resid=48"),                         # more than 256 column tiles: two per workgroup
    ("wide-residual", 1, 5, "resid=48")])
def test_residual_projections_with_the_norm_included(torch_mod, shape_name, B, k, tune):
    """O and down with complete sums, residual add and norm weights in their epilogue, the norm's factor
    applied by the projections behind them: row counts on the kernel's edges, ragged and full row tiles,
    every way the packed matrix can cut the contraction, one and two column tiles per workgroup.  Every
    sequence against its own oracle step."""
    import dataclasses
    shape = (dataclasses.replace(SHAPES["tiny"], name="wide-residual", n_layers=2, d_model=4128, n_heads=2, ffn=112, vocab=300)
             if shape_name == "wide-residual" else SHAPES[shape_name])
    # 2 heads on a width of 4128: logits of std 1.3 out of very few keys, on which a key or value moved by one
    # bf16 step shows more than elsewhere (the split projections with norm launches: 1.0e-3 at k = 2, 5.1e-3 at
    # k = 5); the bar stated for all logits holds
    tol = gc.LOGIT_TOL if shape_name == "wide-residual" else gc.LOGIT_TIGHT
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=4), B, k, tune, tol)


@pytest.mark.parametrize("shape_name,B,k,ctxs", [
    ("tiny", 1, 6, [0]),                   # 49 rows: a last query tile of one row, nothing cached
    ("small128", 2, 7, [31, 700]),         # 64 rows: two full pairs of query tiles, cut over the key axis
    ("gqa128", 3, 7, [1, 64, 333]),
    ("gqa-small", 40, 8, "ragged"),        # 320 x 3 workgroups of two tiles would not fit the chip: three tiles
])
def test_query_tiles_per_workgroup_of_long_blocks(torch_mod, shape_name, B, k, ctxs):
    """Blocks beyond 48 rows on both sides of the rule that gives a workgroup two or three query tiles; every
    sequence against its own oracle step."""
    shape = SHAPES[shape_name]
    if ctxs == "ragged":
        ctxs = [(37 * (b + 1)) % 220 for b in range(B)]
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=6), B, k, None, gc.LOGIT_TIGHT, ctxs=ctxs, capacity=736)


@pytest.mark.parametrize("cut", ["2:0:0:1:0", "0:3:0:0:1", "0:0:4:1:0", "0:0:0:9:1", "1:1:1:0:0", "1:1:1:0:2", "2:0:0:1:2"])
def test_row_cuts_of_split_contractions_give_the_same_bits(torch_mod, cut):
    """As the test with contractions that are never split, at 1024 wide (32 and 43 contraction tiles): 288 rows with the many-row
    kernel forced, where its planner takes two partial sums for QKV, O and down.  A forced cut keeps the partial sums of the default
    one, so logits, indices and accepted counts are equal bit for bit."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES["gqa128"]
    w = all_weights(shape, seed=6)
    B, k = 8, 5
    spec = lo.paper_layout(k)
    L = spec.n_rows
    toks = np.random.default_rng(14).integers(0, shape.vocab, size=(B, L)).astype(np.int32)
    om = gc.oracle_model(shape, w)
    okvs = [gc.synthetic_oracle_kv(om, seed=80 + b, ctx=9 * b + 4, std=0.5) for b in range(B)]
    got = []
    for tune in ("wide=1", "wide=1,widecut=" + cut):
        gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=L, tune=tune)
        cache = gm.kv_cache(B, 160)
        for b in range(B):
            gc.upload_oracle_kv(torch, cache, b, okvs[b])
        out = _run_step(torch, gm, cache, spec, toks, batch=B)
        got.append((out.logits.cpu().numpy().copy(), out.argmax.cpu().numpy().copy(), out.accepted_len.cpu().numpy().copy()))
    for x, y in zip(*got):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("shape_name", ["small128", "gqa128"])  # contractions of 8 and of 32 tiles (two partial sums)
def test_row_cuts_of_the_many_row_kernel_give_the_same_bits(torch_mod, shape_name):
    """288 rows of models whose projections would run in passes, with the many-row kernel forced: every cut of the rows gives the
    logits of the default one bit for bit."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES[shape_name]
    w = all_weights(shape, seed=5)
    spec = lo.paper_layout(5)
    toks = np.random.default_rng(13).integers(0, shape.vocab, size=(8, spec.n_rows)).astype(np.int32)

    def logits(tune):
        gm = gc.make_gpu_model(shape, w, max_batch=8, max_rows=spec.n_rows, tune=tune)
        return _run_step(torch, gm, gm.kv_cache(8, 160), spec, toks, batch=8).logits.cpu().numpy()

    ref = logits("wide=1")
    assert not np.array_equal(ref, logits("wide=0"))  # (another order of sums: the kernel is the one that was forced)
    for cut in ("2:0:0:1:0", "0:3:0:0:0", "0:3:0:0:1", "0:1:3:0:1", "0:0:4:1:0", "0:0:0:9:1", "1:1:1:0:2", "2:0:0:1:2"):
        assert np.array_equal(ref, logits("wide=1,widecut=" + cut)), cut


def test_forced_cut_leaves_no_tail(torch_mod):
    """widecut= and widetail= together, the many-row kernel forced: the forced cut has no piece cut over the contraction, i.e. the
    logits are those of the default cut without tails, bit for bit; at another row count the forced tail still applies.  Where the kernel
    is not forced and these projections run in passes, neither form of widetail= changes a bit."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES["gqa128"]
    w = all_weights(shape, seed=6)
    spec = lo.paper_layout(5)
    toks = np.random.default_rng(14).integers(0, shape.vocab, size=(8, spec.n_rows)).astype(np.int32)

    def logits(B, tune):
        gm = gc.make_gpu_model(shape, w, max_batch=8, max_rows=spec.n_rows, tune=tune)
        return _run_step(torch, gm, gm.kv_cache(B, 160), spec, toks[:B], batch=B).logits.cpu().numpy()

    assert np.array_equal(logits(8, "wide=1,widecut=2:0:0:1:0,widetail=5:3"), logits(8, "wide=1,widetail=0"))
    assert not np.array_equal(logits(7, "wide=1,widecut=2:0:0:1:0,widetail=5:3"), logits(7, "wide=1,widetail=0"))
    passes = logits(8, None)
    assert np.array_equal(logits(8, "widetail=0"), passes) and np.array_equal(logits(8, "widetail=5:3"), passes)


@pytest.mark.parametrize("d,B,k", [(2080, 1, 1), (2080, 3, 3), (3104, 1, 5), (4096, 2, 3), (4128, 1, 4), (8192, 1, 5)])
def test_norm_of_a_row_shared_by_workgroups(torch_mod, d, B, k):
    """Up to 48 rows of models wider than 2048: residual add and norm in workgroups of 1024 columns, the row's factor
    made of their 3 to 8 sums of squares by the projections behind.  Widths with a last workgroup of 32 to 1024 columns; 4, 16,
    25, 32, 36 and 48 rows (all row tiles, ragged last ones); the form with the norm inside the projection is off.  Against the
    oracle."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["tiny"], name="shared-rows", n_layers=2, d_model=d, n_heads=2, ffn=112, vocab=300)
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=12), B, k, "resid=0", gc.LOGIT_TOL)


@pytest.mark.parametrize("shape_name,B,k,order", [("gqa-small", 33, 3, "up"), ("gqa-small", 40, 4, "up"), ("gqa-small", 64, 3, "down"), ("gqa-small", 64, 8, "mixed"),
                                                  ("gqa-small", 65, 4, "mixed"), ("gqa-small", 33, 3, "equal"), ("gqa128", 17, 8, "mixed")])
def test_workgroups_assigned_by_length(torch_mod, shape_name, B, k, order):
    """Batches with more attention workgroups than CUs: 264 to 512 (the last places share a CU with the first), more
    (longest first), 64 sequences and one more than are ordered; lengths ascending, descending, mixed with equal ones, all
    equal, some empty.  Every sequence against its own oracle step."""
    lens = {"up": [9 * b for b in range(B)], "down": [9 * (B - b) for b in range(B)], "mixed": [(211 * (b // 2)) % 500 for b in range(B)],
            "equal": [77] * B}[order]
    _batched_step_vs_oracle(torch_mod, SHAPES[shape_name], all_weights(SHAPES[shape_name], seed=13), B, k, "attn=0", gc.LOGIT_TIGHT, ctxs=lens, capacity=800)


@pytest.mark.parametrize("heads,kv_heads,B,k", [(24, 6, 21, 1), (20, 20, 25, 4), (20, 4, 14, 6), (56, 8, 9, 4)])
def test_workgroups_by_length_where_heads_do_not_divide_the_chip(torch_mod, heads, kv_heads, B, k):
    """480 to 504 workgroups of 20, 24 or 56 heads: those beyond 256 round up to more places than have a partner.  One to
    three query tiles, ascending lengths.  Against the oracle."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["tiny"], name="odd-heads", n_heads=heads, n_kv_heads=kv_heads, vocab=300)
    lens = [(9 * b) if b != B // 2 else 700 for b in range(B)]
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=15), B, k, "attn=0", gc.LOGIT_TIGHT, ctxs=lens, capacity=736)


@pytest.mark.parametrize("shape_name,B,k,order", [("gqa-small", 16, 5, "ragged"), ("gqa-small", 20, 4, "one-long"), ("gqa-small", 32, 5, "ragged"),
                                                  ("gqa-small", 11, 8, "ragged"), ("gqa-small", 31, 5, "equal"), ("small128", 33, 4, "one-long"),
                                                  ("gqa128", 17, 5, "ragged"), ("gqa128", 16, 7, "one-long"), ("small128", 64, 3, "one-long"),
                                                  ("gqa-small", 33, 1, "one-long"), ("gqa-small", 48, 5, "ragged"), ("gqa-small", 63, 3, "one-long")])
def test_keys_of_a_batch_cut_by_length(torch_mod, shape_name, B, k, order):
    """Batches whose workgroups are dealt out by length: sequences in one to sixteen parts, as many slots as the batch
    needs and some left over, empty sequences beside 700 positions, equal lengths (no cut), one to three query tiles, two query
    groups, heads of 64 and 128, more sequences than a workgroup per CU allows (one slot to spare).  Against the oracle, and three steps in a
    row give the same bits (the parts are merged in part order by whoever ends last)."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES[shape_name]
    w = all_weights(shape, seed=14)
    lens = {"ragged": [(67 * b * b) % 701 for b in range(B)], "one-long": [0, 5] + [31 + b for b in range(B - 3)] + [703], "equal": [640] * B}[order]
    _batched_step_vs_oracle(torch, shape, w, B, k, "attn=0", gc.LOGIT_TIGHT, ctxs=lens, capacity=736)
    spec = lo.paper_layout(k)
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=spec.n_rows, tune="attn=0")
    om = gc.oracle_model(shape, w)
    cache = gm.kv_cache(B, 736)
    for b, c in enumerate(lens):
        gc.upload_oracle_kv(torch, cache, b, gc.synthetic_oracle_kv(om, seed=70 + b, ctx=c, std=0.5))
    toks = np.random.default_rng(16).integers(0, shape.vocab, size=(B, spec.n_rows)).astype(np.int32)
    got = [_run_step(torch, gm, cache, spec, toks, batch=B).logits.cpu().numpy().copy() for _ in range(3)]
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])


@pytest.mark.parametrize("shape_name,B,rows,order", [("gqa-small", 9, 112, "one-long"), ("gqa-small", 6, 97, "ragged"), ("gqa-small", 24, 112, "ragged"),
                                                     ("gqa-small", 12, 130, "equal"), ("gqa128", 5, 200, "one-long")])
def test_prompt_chunks_of_a_batch_dealt_out_by_length(torch_mod, shape_name, B, rows, order):
    """Prompt chunks (three to seven query groups) of several sequences behind contexts of 0 to 700 positions: keys cut by length and
    merged per query group, left-over slots, more workgroups than fit at once, equal lengths.  The keys and values that
    the second layer stores, i.e. what the first layer's attention made of the chunk, against the oracle's prefill."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES[shape_name]
    w = all_weights(shape, seed=20)
    lens = {"ragged": [(97 * b * b) % 701 for b in range(B)], "one-long": [9 * b for b in range(B - 1)] + [700], "equal": [600] * B}[order]
    lens[B // 2] = 680
    spec = lo.prefill_layout(rows)
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=rows, max_ctx=1024)
    om = gc.oracle_model(shape, w)
    cache = gm.kv_cache(B, 928)
    okvs = [gc.synthetic_oracle_kv(om, seed=30 + b, ctx=c, std=0.5) for b, c in enumerate(lens)]
    for b in range(B):
        gc.upload_oracle_kv(torch, cache, b, okvs[b])
    toks = np.random.default_rng(21).integers(0, shape.vocab, size=(B, rows)).astype(np.int32)
    gm.prefill(torch.from_numpy(toks).cuda(), gm.layout(spec), cache)
    torch.cuda.synchronize()
    assert gm.device_faults() == 0
    for b, c in enumerate(lens):
        so.prefill(om, okvs[b], toks[b])
        gk, gv = gc.download_kv_rows(cache, 1, b, c, c + rows)
        gc.assert_bf16_close(gk, okvs[b].k[1][c:], f"seq {b} K", min_same=0.9)
        gc.assert_bf16_close(gv, okvs[b].v[1][c:], f"seq {b} V", min_same=0.9)


@pytest.mark.parametrize("shape_name,B,rows,tune,tuned", [
    ("tiny", 1, 9, None, False), ("gqa-small", 2, 40, "qkv=6:2", False), ("gqa128", 1, 70, "qkv=8:1", False), ("small128", 3, 50, "qkv=6:1", False),
    ("gqa-small", 1, 150, "wide=1", False), ("gqa128", 2, 130, "wide=1,wideks=2", False), ("small128", 1, 330, "wide=1,wideks=4", False),
    ("tiny", 2, 300, "qkv=6:1", False), ("gqa128", 1, 200, "wide=1", True), ("gqa-small", 2, 161, "wide=1,wideks=2", True)])
def test_last_layer_of_a_prompt_chunk_without_queries(torch_mod, shape_name, B, rows, tune, tuned):
    """The last layer's projection starts at the first key's weight tile (few rows: at the group of tiles that holds it, which need
    not start there): that layer's keys and values of chunks with one, two and many query tiles and passes, in both projection
    kernels, with partial sums, in tuned contexts (which leave that launch as it is planned) too, against the oracle's prefill; the layer in front keeps its own."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES[shape_name].with_layers(2)
    w = all_weights(shape, seed=23)
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=rows, max_ctx=512, tune=tune)
    if tuned:
        gm.tune_rows(B * rows)
    om = gc.oracle_model(shape, w)
    cache = gm.kv_cache(B, 512)
    lens = [13 + 50 * b for b in range(B)]
    okvs = [gc.synthetic_oracle_kv(om, seed=40 + b, ctx=c, std=0.5) for b, c in enumerate(lens)]
    for b in range(B):
        gc.upload_oracle_kv(torch, cache, b, okvs[b])
    toks = np.random.default_rng(24).integers(0, shape.vocab, size=(B, rows)).astype(np.int32)
    gm.prefill(torch.from_numpy(toks).cuda(), gm.layout(lo.prefill_layout(rows)), cache)
    torch.cuda.synchronize()
    assert gm.device_faults() == 0
    for b, c in enumerate(lens):
        so.prefill(om, okvs[b], toks[b])
        for l in range(2):
            gk, gv = gc.download_kv_rows(cache, l, b, c, c + rows)
            gc.assert_bf16_close(gk, okvs[b].k[l][c:], f"layer {l} seq {b} K", min_same=0.9)
            gc.assert_bf16_close(gv, okvs[b].v[l][c:], f"layer {l} seq {b} V", min_same=0.9)


@pytest.mark.parametrize("shape_name,rows,ctxs,tune", [
    ("small128", 36, [500], "attn=1000000"),   # one launch per layer
    ("small128", 36, [700], "attn=0"),         # keys cut over workgroups
    ("gqa-small", 25, "ragged", "attn=0"),     # a batch dealt out and cut by length
    ("gqa128", 70, [700, 90], None),
    ("gqa-small", 193, "ragged", None)])       # attn_rows_kernel
def test_large_values_of_a_steep_softmax_stay_finite(torch_mod, shape_name, rows, ctxs, tune):
    """Cached values of 2^121 to 2^122 and keys whose scores spread over some tens: no weight of the softmax may be above 1 on the way, or
    the sums of a wave's chunks overflow where the output does not.  The first layer's attention output of every row against the
    oracle's; bars relative to the largest (2^-17 per operand of scores up to some tens in the exponent)."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES[shape_name].with_layers(2)
    w = all_weights(shape, seed=27)
    if ctxs == "ragged":
        ctxs = [(151 * b) % 690 for b in range(11)] + [700]
    B, cap = len(ctxs), 1024
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=rows, max_ctx=cap, tune=tune)
    om = gc.oracle_model(shape, w)
    okvs = [gc.synthetic_oracle_kv(om, seed=50 + b, ctx=c, std=16.0) for b, c in enumerate(ctxs)]
    cache = gm.kv_cache(B, cap)
    for b, okv in enumerate(okvs):
        okv.v[0] = gc.bits_to_f64(gc.f32_to_bf16_bits((2.0 ** 121 * (1.0 + np.minimum(np.abs(okv.v[0]), 15.0) / 16.0)).astype(np.float32)))
        gc.upload_oracle_kv(torch, cache, b, okv)
    toks = np.random.default_rng(28).integers(0, shape.vocab, size=(B, rows)).astype(np.int32)
    spec = lo.prefill_layout(rows)
    gm.prefill(torch.from_numpy(toks).cuda(), gm.layout(spec), cache)
    torch.cuda.synchronize()
    hd = shape.n_heads * shape.head_dim
    out = gc.decode_planes(gm.debug_buffer("attn_out"), B * rows, hd).reshape(B, rows, hd)
    for b, okv in enumerate(okvs):
        trace = []
        so.block_forward_cached(om, okv, toks[b].astype(np.int64), spec.is_mask.astype(bool), trace=trace)
        ref = trace[0]["attn_out"].reshape(rows, hd)
        assert np.abs(out[b] - ref).max() < 2e-3 * max(np.abs(ref).max(), 1.0), b


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_a_key_that_is_no_number_shows_through_the_merge(torch_mod, value):
    """One sequence of a batch, long enough to be cut into parts, with one cached key element that is NaN or infinite: a score of the
    softmax is no number then, so every logit of that sequence is NaN (as where one workgroup takes all keys), and
    the other sequences' logits keep their bits."""
    torch = torch_mod
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES["gqa-small"]
    B, k, long_one = 20, 4, 19
    lens = [5 + b for b in range(B - 1)] + [703]
    spec = lo.paper_layout(k)
    gm = gc.make_gpu_model(shape, all_weights(shape, seed=14), max_batch=B, max_rows=spec.n_rows, tune="attn=0")
    om = gc.oracle_model(shape, all_weights(shape, seed=14))
    cache = gm.kv_cache(B, 736)
    for b, c in enumerate(lens):
        gc.upload_oracle_kv(torch, cache, b, gc.synthetic_oracle_kv(om, seed=70 + b, ctx=c, std=0.5))
    cache.len.copy_(torch.tensor(lens, dtype=torch.int32))
    cache.set_len_bound(max(lens))
    toks = np.random.default_rng(17).integers(0, shape.vocab, size=(B, spec.n_rows)).astype(np.int32)
    clean = _run_step(torch, gm, cache, spec, toks, batch=B).logits.cpu().numpy().copy()
    cache.k_view()[0, long_one, :, 333, 0] = value
    got = _run_step(torch, gm, cache, spec, toks, batch=B).logits.cpu().numpy()
    assert np.isfinite(clean).all()
    assert np.isnan(got[long_one]).all()
    others = [b for b in range(B) if b != long_one]
    assert np.array_equal(got[others], clean[others])


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("shape_name,rows,ctxs", [("64 heads", 257, [400]), ("gqa-small", 193, "ragged")])
def test_a_key_that_is_no_number_shows_in_long_blocks(torch_mod, shape_name, rows, ctxs, value):
    """attn_rows_kernel, one workgroup for all keys and parts merged by whoever ends last, with one cached key element that is NaN or
    infinite: the attention output of every row and head of that sequence is NaN where the softmax is (infinite keys: unless both
    halves of the query's element are negative, when the key has no weight), and the other sequences' keep their bits."""
    torch = torch_mod
    import dataclasses
    from paper_2402_11809_amd import layout as lo
    shape = SHAPES["gqa-small"].with_layers(2)
    if shape_name == "64 heads":
        shape = dataclasses.replace(shape, n_heads=64, n_kv_heads=8)
    if ctxs == "ragged":
        ctxs = [(151 * b) % 690 for b in range(11)] + [700]
    B, hd, one = len(ctxs), shape.n_heads * shape.head_dim, len(ctxs) - 1
    w = all_weights(shape, seed=8)
    gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=rows, max_ctx=1024)
    om = gc.oracle_model(shape, w)
    cache = gm.kv_cache(B, 1024)
    for b, c in enumerate(ctxs):
        gc.upload_oracle_kv(torch, cache, b, gc.synthetic_oracle_kv(om, seed=30 + b, ctx=c, std=0.5))
    toks = torch.from_numpy(np.random.default_rng(11).integers(0, shape.vocab, size=(B, rows)).astype(np.int32)).cuda()

    def attention():
        gm.prefill(toks, gm.layout(lo.prefill_layout(rows)), cache)
        torch.cuda.synchronize()
        return gc.decode_planes(gm.debug_buffer("attn_out"), B * rows, hd).reshape(B, rows, shape.n_heads, shape.head_dim)

    clean = attention()
    cache.k_view()[0, one, :, 333, 0] = value
    got = attention()
    q = gc.bits_to_f64(gm.debug_buffer("q")[: 2 * B * rows * hd]).reshape(2, B, shape.n_heads, rows, shape.head_dim)
    hi, lo_ = (q[plane, one, :, :, 0].T for plane in (0, 1))  # [row, head]
    assert np.isfinite(clean).all()
    hit = np.ones_like(hi, dtype=bool) if np.isnan(value) else ~((hi < 0) & (lo_ < 0))
    assert hit.any() and (np.isnan(value) or not hit.all())
    assert np.isnan(got[one][hit]).all() and np.isfinite(got[one][~hit]).all()
    assert np.array_equal(got[:one], clean[:one])


@pytest.fixture(scope="module")
def one_layer_7b(torch_mod):
    """logits(tune, tuned): 288 rows of one layer of 7B width, from a new context each time."""
    import dataclasses
    from paper_2402_11809_amd import layout as lo
    shape = dataclasses.replace(SHAPES["7b"], name="7b-1l", n_layers=1, vocab=300)
    w = all_weights(shape, seed=18, threads=16)
    B, spec = 8, lo.paper_layout(5)
    toks = np.random.default_rng(19).integers(0, shape.vocab, size=(B, spec.n_rows)).astype(np.int32)

    def logits(tune=None, tuned=False):
        gm = gc.make_gpu_model(shape, w, max_batch=B, max_rows=spec.n_rows, max_ctx=128, tune=tune)
        if tuned:
            gm.tune_rows(B * spec.n_rows)
        return _run_step(torch_mod, gm, gm.kv_cache(B, 64), spec, toks, batch=B).logits.cpu().numpy()

    return logits


def test_tuned_contexts_keep_the_planned_tail(one_layer_7b):
    """288 rows at 7B width, where the planner cuts the last pieces of gate / up over the contraction (the logits differ from
    those of a context without such pieces): measured, that form and the plan without it are within a few percent of each other, so
    space_tune_rows must not choose between them by the clock.  Six tuned contexts give the untuned one's bits, and all are
    within 1e-3 of the form without (the bar of the other tuning test)."""
    plain, without = one_layer_7b(), one_layer_7b("widetail=0")
    assert not np.array_equal(plain, without) and np.abs(plain - without).max() < 1e-3
    for _ in range(6):
        assert np.array_equal(one_layer_7b(tuned=True), plain)


def test_tails_take_no_memory_of_their_own(torch_mod):
    """A context of 288 rows at 7B width, whose partial sums of split contractions have room for those of the tails: as much device memory
    as one without tails (allocations are whole pages of 2 MB)."""
    torch = torch_mod
    import dataclasses
    shape = dataclasses.replace(SHAPES["tiny"], name="7b-wide", n_layers=1, d_model=4096, n_heads=32, head_dim=128, ffn=256, vocab=300)
    w = all_weights(shape, seed=22)

    def free():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    models, taken = [], []
    for tune in (None, "widetail=0", None):  # the first one also pays for what the process allocates once
        before = free()
        models.append(gc.make_gpu_model(shape, w, max_batch=8, max_rows=36, max_ctx=128, tune=tune))
        taken.append(before - free())
    assert abs(taken[2] - taken[1]) <= 4 << 20, taken


def test_forced_tail_holds_where_rows_are_tuned(one_layer_7b):
    """SPACE_TUNE widetail=P:N is applied whether or not the row count was tuned (nothing else is 10 % ahead there: previous
    test)."""
    plain, forced = one_layer_7b(), one_layer_7b("widetail=6:2")
    assert not np.array_equal(plain, forced) and np.abs(plain - forced).max() < 1e-3
    assert np.array_equal(one_layer_7b("widetail=6:2", tuned=True), forced)


@pytest.mark.parametrize("vocab", [1000, 32000])  # partials per row: fewer than a wave's lanes, several per lane
@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 48, 49, 96])
def test_argmax_of_every_row_at_the_edges_of_the_rows_per_wave(torch_mod, rows, vocab):
    """The verification merges one, two or three rows per wave and trip (16 waves): the argmax of every row of
    two sequences is that of its own logits (lowest id of equal ones), the extra token that of the first row."""
    torch = torch_mod
    import dataclasses
    from paper_2402_11809_amd import binding, layout as lo
    shape = dataclasses.replace(SHAPES["tiny"], vocab=vocab, n_layers=1)
    B = 2
    gm = gc.make_gpu_model(shape, all_weights(shape, seed=3), max_batch=B, max_rows=rows, max_ctx=128)
    spec = lo.first_step_layout(rows - 1)
    assert spec.n_rows == rows
    cache = gm.kv_cache(B, 128)
    toks = np.random.default_rng(rows).integers(0, vocab, size=(B, rows)).astype(np.int32)
    out = binding.StepOut(gm, B, rows, max(rows - 1, 1))
    gm.step(torch.from_numpy(toks).cuda(), gm.layout(spec), cache, out)
    torch.cuda.synchronize()
    want = out.logits.cpu().numpy().reshape(B, rows, vocab).argmax(2)
    assert np.array_equal(out.argmax.cpu().numpy().reshape(B, rows), want)
    assert out.bonus.cpu().numpy().tolist() == want[:, 0].tolist()
    assert out.accepted_len.cpu().numpy().tolist() == [0, 0]


@pytest.mark.parametrize("shape_name,k,ctx", [("tiny", 1, 703), ("tiny", 3, 736), ("tiny", 3, 737), ("gqa-small", 4, 704), ("gqa-small", 4, 705)])
def test_attention_of_64_element_heads_around_its_line(torch_mod, shape_name, k, ctx):
    """Heads of 64 elements take the one-launch attention up to 24 chunks of 32 keys (the cached ones and the
    block's), the cut over the key axis beyond: one and two query tiles on both sides of the line against the oracle."""
    shape = SHAPES[shape_name]
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=8), 1, k, None, gc.LOGIT_TIGHT, ctxs=[ctx], capacity=768)


@pytest.mark.parametrize("B", [32, 33])
def test_one_tile_attention_on_both_sides_of_a_workgroup_per_cu(torch_mod, B):
    """Blocks of one query tile take the one-launch attention up to 256 (sequence, head) pairs and the cut over the key
    axis beyond: 32 and 33 sequences of 8 heads with short ragged contexts against the oracle."""
    shape = SHAPES["gqa-small"]
    _batched_step_vs_oracle(torch_mod, shape, all_weights(shape, seed=9), B, 1, None, gc.LOGIT_TIGHT)

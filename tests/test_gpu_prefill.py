"""Context prefill through the C ABI (chunked chain passes) against the oracle's single
causal pass: committed K/V, context counters and the first greedy token."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.model import argmax_low
from gpu_util import dev_i32, read_cache

pytestmark = pytest.mark.gpu

KV_TOL = 3e-2         # same bar as the step tests put on a pass' K/V rows
MARGIN = 6e-2


@pytest.fixture(scope="module")
def bita():
    import paper_2401_12522_amd as b
    b.lib()
    return b


def _oracle_causal(om, toks):
    """K/V and last-row logits of one causal pass over toks from an empty cache."""
    cfg = om.cfg
    n = len(toks)
    ck = [np.zeros((0, cfg.n_kv_heads, cfg.head_dim)) for _ in range(cfg.n_layers)]
    cv = [np.zeros((0, cfg.n_kv_heads, cfg.head_dim)) for _ in range(cfg.n_layers)]
    vis = [list(range(r + 1)) for r in range(n)]
    logits, k, v = oracle.forward_rows(om, list(toks), [0] * n, [-1] * n, list(range(n)), vis, ck, cv)
    return k, v, logits[n - 1]


def _margin(row):
    s = np.sort(row)
    return s[-1] - s[-2]


@pytest.mark.parametrize("cfg_name,n_ctx,chunk", [("tiny", 150, 64), ("tiny_gqa", 150, 256), ("tiny_gqa", 97, 17),
                                                  ("tiny", 600, 512)])      # 512 rows: the largest template
def test_prefill_chunks_match_one_causal_pass(bita, cfg_name, n_ctx, chunk):
    cfg = synth.get_config(cfg_name)
    w = synth.SynthWeights(cfg, seed=3)
    om = oracle.OracleModel(cfg, w)
    smax = 256 if n_ctx <= 256 else 640
    model = bita.Model(cfg, w, max_pos=smax + 64)
    kv = bita.KVState(cfg, cfg.n_layers, 1, smax, chunk)
    ctx = synth.random_context(cfg.vocab, n_ctx, 11)
    nxt = bita.prefill(model, kv, 0, dev_i32(ctx[None]), chunk)
    torch.cuda.synchronize()
    assert int(kv.ctx_len[0]) == n_ctx
    k, v, last = _oracle_causal(om, ctx)
    gk, gv = read_cache(kv)
    for l in range(cfg.n_layers):
        assert gk[l].shape == k[l].shape
        assert np.abs(gk[l] - k[l]).max() <= KV_TOL
        assert np.abs(gv[l] - v[l]).max() <= KV_TOL
    # slots past the context stay untouched (the cache starts zeroed)
    assert not kv.k_cache[:, 0, :, n_ctx:].any() and not kv.v_cache[:, 0, :, n_ctx:].any()
    if _margin(last) > MARGIN:
        assert int(nxt[0]) == argmax_low(last)
    else:
        assert 0 <= int(nxt[0]) < cfg.vocab


def test_prefill_ragged_batch_in_two_calls(bita):
    """Three sequences of different lengths (one empty), filled by two calls: the second call
    appends to what the first committed.  Each sequence equals its own causal pass."""
    cfg = synth.get_config("tiny_gqa")
    w = synth.SynthWeights(cfg, seed=5)
    om = oracle.OracleModel(cfg, w)
    smax, chunk, B = 256, 48, 3
    model = bita.Model(cfg, w, max_pos=smax + 64)
    kv = bita.KVState(cfg, cfg.n_layers, B, smax, chunk)
    lens = [131, 37, 0]
    first = [60, 37, 0]                                  # tokens handed over by the first call
    ctxs = [synth.random_context(cfg.vocab, max(n, 1), 40 + b)[:n] for b, n in enumerate(lens)]

    def padded(parts):
        width = max(max(len(p) for p in parts), 1)
        out = np.full((B, width), -7, np.int32)           # padding is never read as a token
        for b, p in enumerate(parts):
            out[b, :len(p)] = p
        return dev_i32(out)
    n1 = bita.prefill(model, kv, 0, padded([c[:f] for c, f in zip(ctxs, first)]), chunk, seq_len=dev_i32(first))
    torch.cuda.synchronize()
    assert kv.ctx_len.cpu().tolist() == first
    rest = [len(c) - f for c, f in zip(ctxs, first)]
    n2 = bita.prefill(model, kv, max(first), padded([c[f:] for c, f in zip(ctxs, first)]), chunk, seq_len=dev_i32(rest))
    torch.cuda.synchronize()
    assert kv.ctx_len.cpu().tolist() == lens
    assert int(n1[2]) == -1 and int(n2[2]) == -1          # an empty sequence has no next token
    assert int(n2[1]) == -1                               # nothing of sequence 1 in the second call
    for b in range(B):
        if lens[b] == 0:
            continue
        k, v, last = _oracle_causal(om, ctxs[b])
        gk, gv = read_cache(kv, b=b)
        for l in range(cfg.n_layers):
            assert np.abs(gk[l] - k[l]).max() <= KV_TOL
            assert np.abs(gv[l] - v[l]).max() <= KV_TOL
        got = int(n2[b]) if rest[b] > 0 else int(n1[b])
        if _margin(last) > MARGIN:
            assert got == argmax_low(last)


@pytest.mark.parametrize("heads,kv_heads,hd,batch,chunk,longest", [
    (8, 1, 128, 3, 40, 155), (16, 2, 64, 3, 64, 250), (32, 1, 64, 2, 33, 99),     # 4 rows a workgroup, 4, 2
    (8, 1, 128, 3, 40, 131), (6, 1, 64, 2, 40, 60),                               # few rows, and heads that do not share tiles: 16
    (64, 8, 64, 40, 48, 90), (64, 8, 128, 36, 33, 60),                            # more workgroups than CUs: four waves
    (4, 4, 128, 3, 40, 131), (4, 4, 64, 70, 33, 90),                              # one head per workgroup: the one row tile alone
    (8, 1, 64, 1, 40, 2000)])                                                     # the keys split between workgroups
def test_the_token_after_a_prompt_is_that_of_passes_that_finish_every_row(bita, heads, kv_heads, hd, batch, chunk, longest):
    """A prefill's last layer goes on with one row per sequence, and attention with the workgroups that hold it.  The
    tokens after all rows of the last chunk, by a pass that finishes them all, are the reference, wherever each sequence ends."""
    cfg = synth.get_config("tiny", n_heads=heads, n_kv_heads=kv_heads, head_dim=hd)
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=6, device="cuda"), max_pos=longest + 64)
    rng = np.random.default_rng(heads + chunk)
    last = longest - (longest - 1) // chunk * chunk                               # rows of the last chunk
    first = longest - last
    toks = dev_i32(rng.integers(0, cfg.vocab, (batch, longest)))
    ends = first + 1 + np.arange(batch) * 5 % last                                # every place of a tile
    kv = bita.KVState(cfg, cfg.n_layers, batch, longest + 8, chunk)
    nxt = bita.prefill(model, kv, 0, toks, chunk, seq_len=dev_i32(ends))
    every = bita.KVState(cfg, cfg.n_layers, batch, longest + 8, chunk)
    if first:
        bita.prefill(model, every, 0, toks[:, :first].contiguous(), chunk)
    every.resize_rows(cfg.n_layers, cfg, last)
    tmpl = bita.TreeTemplate(np.arange(last, dtype=np.int32) - 1, np.zeros(last, np.uint8), last, cfg.n_mask)
    buf = bita.StepBuffers(model, tmpl, batch, 1, want_logits=True)
    buf.token.copy_(toks[:, first:])
    bita.verify_step(model, every, first, tmpl, buf, batch)
    torch.cuda.synchronize()
    assert kv.ctx_len.cpu().tolist() == ends.tolist()
    rows = torch.tensor(ends - first - 1, device="cuda")
    logits = buf.logits[torch.arange(batch, device="cuda"), rows]
    assert torch.isfinite(logits).all()
    two = torch.topk(logits, 2).values
    # (the two passes' sums are ordered differently: 4e-5 of a logit's size between them, and the cache's stored rows a unit here and there)
    clear = (two[:, 0] - two[:, 1]) > 1e-2 * logits.abs().amax(1)
    assert bool(clear.any())
    assert torch.equal(nxt[clear], torch.argmax(logits, 1)[clear].int())


def test_prefill_rejects_what_does_not_fit(bita):
    cfg = synth.get_config("tiny")
    w = synth.SynthWeights(cfg, seed=1)
    model = bita.Model(cfg, w, max_pos=96)
    kv = bita.KVState(cfg, cfg.n_layers, 1, 64, 32)
    toks = dev_i32(synth.random_context(cfg.vocab, 80, 2)[None])
    with pytest.raises(bita.BitaError) as e:
        bita.prefill(model, kv, 0, toks, 32)              # 80 tokens into 64 slots
    assert e.value.code == -3
    with pytest.raises(bita.BitaError) as e:
        bita.prefill(model, kv, 0, toks[:, :40].contiguous(), 33)   # scratch holds 32 rows
    assert e.value.code == -1
    # an empty context is a no-op, not an error
    nxt = bita.prefill(model, kv, 0, torch.zeros((1, 0), dtype=torch.int32, device="cuda"), 32)
    torch.cuda.synchronize()
    assert int(nxt[0]) == -1
    assert int(kv.ctx_len[0]) == 0 and not kv.k_cache.any()


def test_prompt_to_tokens_on_the_device_alone(bita):
    """The whole decoder with no oracle data on the device: prefill of the full prompt gives the
    first token, then the first step runs with no candidates (Algorithm 1, t = 1: only the root
    and its mask rows are live) and later steps draft for themselves.  The emitted stream is the
    oracle's autoregressive greedy stream wherever its top-2 margin is decisive."""
    cfg = synth.get_config("tiny")
    tin = synth.attach_mask_groups(synth.random_tree(8, 3, 0), [0], cfg.n_mask)
    w = synth.SynthWeights(cfg, seed=0)
    om = oracle.OracleModel(cfg, w)
    d = oracle.tree.derive_template(tin.parent, tin.is_mask, tin.n_mask)
    smax, steps = 256, 12
    model = bita.Model(cfg, w, max_pos=smax + 64)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, tin.n_mask)
    kv = bita.KVState(cfg, cfg.n_layers, 1, smax, max(tmpl.rows, 32))
    ctx = synth.random_context(cfg.vocab, 64, 0)
    # oracle: greedy stream and margins, one token per pass
    ck, cv = oracle.decode.prefill(om, ctx)
    ref, margins = [], []
    last = int(ctx[-1])
    for _ in range(steps * (d.tree_depth + 1) + 2):
        lg, k, v = oracle.forward_rows(om, [last], [0], [-1], [ck[0].shape[0]], [[0]], ck, cv)
        ck, cv = oracle.compact_kv(ck, cv, k, v, [0])
        last = argmax_low(lg[0])
        ref.append(last)
        margins.append(_margin(lg[0]))
    # device: prompt -> first token -> steps
    first = bita.prefill(model, kv, 0, dev_i32(ctx[None]), 32)
    emitted = [int(first[0])]
    kv.resize_rows(cfg.n_layers, cfg, tmpl.rows)
    buf = bita.StepBuffers(model, tmpl, 1, d.kmax)
    buf.bonus.copy_(first)
    buf.next_shift[0] = cfg.n_mask                       # t = 1: no candidates yet
    lens = []
    for t in range(steps):
        hint = len(ctx) + t * (d.tree_depth + 1)
        bita.decode_step(model, kv, hint, tmpl, buf, 1, buf.bonus, buf.topk_ids, buf.next_group, buf.next_shift)
        torch.cuda.synchronize()
        na = int(buf.n_acc[0])
        if t == 0:
            assert na == 1 and buf.token[0, 1:tmpl.n_tree].cpu().tolist() == [-1] * (tmpl.n_tree - 1)
        lens.append(na)
        emitted.extend(buf.emitted[0, :na].cpu().tolist())
    low = [i for i in range(len(emitted)) if margins[i] <= MARGIN]
    upto = low[0] if low else len(emitted)
    assert upto >= 8, "seed gives an early near-tie; pick another"
    assert emitted[:upto] == ref[:upto]
    assert int(kv.ctx_len[0]) == len(ctx) + sum(lens)


def test_prefill_and_first_step_replay_from_one_graph(bita):
    """bita_prefill allocates nothing and never waits for the stream once the model holds its
    chain templates: prefill of the prompt and the first step are captured into one HIP graph
    and replayed on reset state three times, with eager work in between; every replay gives the
    eager run's bits, and the tokens are the oracle's greedy ones where its margin is decisive."""
    cfg = synth.get_config("tiny_gqa")
    tin = synth.attach_mask_groups(synth.random_tree(8, 3, 0), [0], cfg.n_mask)
    w = synth.SynthWeights(cfg, seed=2, norm_std=0.3, prefix_std=1.0)
    om = oracle.OracleModel(cfg, w)
    d = oracle.tree.derive_template(tin.parent, tin.is_mask, tin.n_mask)
    smax, chunk, n_ctx = 256, 32, 75                     # two full chunks and a ragged one of 11 rows
    model = bita.Model(cfg, w, max_pos=smax + 64)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, tin.n_mask)
    kv = bita.KVState(cfg, cfg.n_layers, 1, smax, chunk)
    kv_step = bita.KVState.__new__(bita.KVState)         # the same memory, laid out for the step's rows
    kv_step.__dict__.update(kv.__dict__)
    kv_step.resize_rows(cfg.n_layers, cfg, tmpl.rows)
    ctx = synth.random_context(cfg.vocab, n_ctx, 5)
    toks = dev_i32(ctx[None])
    ws = bita.prefill_workspace(model, 1, chunk)
    first = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    buf = bita.StepBuffers(model, tmpl, 1, d.kmax, want_logits=True)
    shift0 = dev_i32([cfg.n_mask])                       # t = 1: no candidates yet

    def reset():
        kv.ctx_len.zero_(); kv.k_cache.zero_(); kv.v_cache.zero_(); first.fill_(-1)

    def run():
        bita.prefill(model, kv, 0, toks, chunk, workspace=ws, next_token=first)
        bita.decode_step(model, kv_step, n_ctx, tmpl, buf, 1, first, buf.topk_ids, None, shift0)

    bita.prefill_prepare(model, n_ctx, chunk)
    reset()
    run()                                                # eager
    torch.cuda.synchronize()
    eager = [first.clone(), buf.logits.clone(), buf.bonus.clone(), kv.k_cache.clone(), kv.ctx_len.clone()]
    assert int(kv.ctx_len[0]) == n_ctx + 1
    graph = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream()
    reset()
    with torch.cuda.stream(st):
        with torch.cuda.graph(graph, stream=st):
            run()
    torch.cuda.synchronize()
    for rep in range(3):
        reset()
        buf.logits.fill_(7.0)
        (torch.ones(1 << 20, device="cuda") * 3).sum().item()   # the program's own eager work between replays
        graph.replay()
        torch.cuda.synchronize()
        got = [first, buf.logits, buf.bonus, kv.k_cache, kv.ctx_len]
        for a, b_ in zip(eager, got):
            assert torch.equal(a, b_), rep
    # against the oracle: the token after the prompt
    _, _, last = _oracle_causal(om, [int(x) for x in ctx])
    if _margin(last) > MARGIN:
        assert int(first[0]) == argmax_low(last)


def test_prefill_on_a_capturing_stream_needs_its_templates(bita):
    """A capturing stream that finds no chain template is refused, not served by an allocation."""
    cfg = synth.get_config("tiny")
    w = synth.SynthWeights(cfg, seed=1)
    model = bita.Model(cfg, w, max_pos=128)
    kv = bita.KVState(cfg, cfg.n_layers, 1, 96, 32)
    toks = dev_i32(synth.random_context(cfg.vocab, 50, 2)[None])
    ws = bita.prefill_workspace(model, 1, 32)
    first = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    bita.prefill(model, kv, 0, toks, 32, workspace=ws, next_token=first)      # eager: creates 32 and 18
    torch.cuda.synchronize()
    kv.ctx_len.zero_()
    graph, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with pytest.raises(bita.BitaError) as e:
        with torch.cuda.stream(st):
            with torch.cuda.graph(graph, stream=st):
                bita.prefill(model, kv, 0, toks, 29, workspace=ws, next_token=first)   # chunks of 29 and 21: unknown
    assert e.value.code == -1 and "bita_prefill_prepare" in str(e.value)
    torch.cuda.synchronize()
    assert int(kv.ctx_len[0]) == 0


@pytest.mark.parametrize("batch,chunk", [(1, 16), (3, 25), (17, 21), (20, 24)])   # 1, 3, 17 and 20 rows behind the last K/V projection
def test_next_token_comes_from_the_last_rows_alone(bita, batch, chunk):
    """Sequences that end in the first, a middle and the last chunk, at a chunk's first and last row, or
    are empty: the greedy token equals the one of a pass that computes every row's logits, and a call
    that asks for no token leaves the same cache."""
    from paper_2401_12522_amd import binding as B
    cfg = synth.get_config("tiny_gqa")
    w = synth.SynthWeights(cfg, seed=8)
    n = 50
    model = bita.Model(cfg, w, max_pos=256)
    lens = [n, 1, 0, chunk, chunk + 1, 2 * chunk - 1, 2 * chunk][:batch] + [(7 * i) % (n + 1) for i in range(max(0, batch - 7))]
    toks = dev_i32(np.random.default_rng(batch).integers(0, cfg.vocab, size=(batch, n)))
    seq = dev_i32(lens) if batch > 1 else None
    kv = bita.KVState(cfg, cfg.n_layers, batch, 128, chunk)
    nxt = bita.prefill(model, kv, 0, toks, chunk, seq_len=seq).cpu().tolist()
    kv0 = bita.KVState(cfg, cfg.n_layers, batch, 128, chunk)
    ws = bita.prefill_workspace(model, batch, chunk)
    B._check(B.lib().bita_prefill(model.handle, B.C.byref(kv0.desc(0)), B._ptr(toks), n, B._ptr(seq), B._ptr(kv0.ctx_len), batch,
                                  chunk, B._ptr(ws), ws.numel(), None, B._stream()))
    torch.cuda.synchronize()
    assert kv0.ctx_len.cpu().tolist() == lens == kv.ctx_len.cpu().tolist()
    assert torch.equal(kv0.k_cache, kv.k_cache) and torch.equal(kv0.v_cache, kv.v_cache)
    chain = bita.TreeTemplate(synth.chain_tree(n), np.zeros(n, np.uint8), n, 0)
    full = bita.KVState(cfg, cfg.n_layers, 1, 128, n)
    buf = bita.StepBuffers(model, chain, 1, 1, want_logits=True)
    for b, len_b in enumerate(lens):
        if len_b == 0:
            assert nxt[b] == -1
            continue
        buf.token.copy_(toks[b:b + 1])
        bita.verify_step(model, full, 0, chain, buf, 1)
        last = buf.logits[0, len_b - 1].cpu().numpy()
        # both sides are within 1e-4 of exact logits (chunks after the first see a bf16 cache: 3e-2)
        assert nxt[b] == argmax_low(last) or _margin(last) < (2e-4 if len_b <= chunk else MARGIN), (b, len_b)


@pytest.mark.parametrize("cfg_name,batch,n", [("tiny", 1, 16), ("tiny_gqa", 1, 21), ("tiny_gqa", 2, 35)])
def test_next_token_behind_a_split_key_axis(bita, cfg_name, batch, n):
    """Chunks of 16 rows on a context long enough that attention splits its keys: the partial sums of the one
    row that goes on are merged, from a workspace that held NaN; token and cache equal those of passes
    that finish every row."""
    from paper_2401_12522_amd import binding as B
    cfg = synth.get_config(cfg_name)
    ctx, chunk = 2300, 16
    P, hd = cfg.n_prompt, cfg.head_dim
    ws_of = lambda rows, at: B.lib().bita_attention_workspace_bytes(batch, rows, cfg.n_heads, hd, at, P)     # noqa: E731
    for at in range(0, n, chunk):
        rows = min(chunk, n - at)                        # more than one split's partial sums (hd + 2 floats a row)
        assert ws_of(rows, ctx + at) >= 2 * batch * cfg.n_heads * rows * (hd + 2) * 4
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=9), max_pos=ctx + 128)
    lens = [n - 5 * b for b in range(batch)]
    rng = np.random.default_rng(n)
    toks = dev_i32(rng.integers(0, cfg.vocab, size=(batch, n)))
    kv = [bita.KVState(cfg, cfg.n_layers, batch, ctx + 64, chunk) for _ in range(2)]
    g = torch.Generator(device="cuda").manual_seed(1)
    for name in ("k_cache", "v_cache"):
        fill = torch.randn(kv[0].k_cache[:, :, :, :ctx].shape, generator=g, device="cuda").to(torch.bfloat16)
        for s in kv:
            getattr(s, name)[:, :, :, :ctx] = fill
    for s in kv:
        s.ctx_len.fill_(ctx)
    ws = bita.prefill_workspace(model, batch, chunk)
    ws.fill_(0xFF)
    nxt = bita.prefill(model, kv[0], ctx, toks, chunk, seq_len=dev_i32(lens), workspace=ws).cpu().tolist()
    last = [None] * batch
    for at in range(0, n, chunk):
        rows = min(chunk, n - at)
        kv[1].resize_rows(cfg.n_layers, cfg, rows)
        chain = bita.TreeTemplate(synth.chain_tree(rows), np.zeros(rows, np.uint8), rows, 0)
        buf = bita.StepBuffers(model, chain, batch, 1, want_logits=True)
        inside = torch.arange(rows, device="cuda")[None] + at < dev_i32(lens)[:, None]
        buf.token.copy_(torch.where(inside, toks[:, at:at + rows], -1))
        bita.verify_step(model, kv[1], ctx + at, chain, buf, batch)
        n_acc = inside.sum(1).to(torch.int32)
        path = torch.arange(rows, dtype=torch.int32, device="cuda").expand(batch, rows).contiguous()
        bita.compact_kv(model, kv[1], ctx + at, buf, batch, path=path, n_acc=n_acc)
        for b in range(batch):
            if at < lens[b] <= at + rows:
                last[b] = buf.logits[b, lens[b] - 1 - at].cpu().numpy()
    torch.cuda.synchronize()
    for b in range(batch):
        assert torch.equal(kv[0].k_cache[:, b, :, :ctx + lens[b]], kv[1].k_cache[:, b, :, :ctx + lens[b]])
        assert torch.equal(kv[0].v_cache[:, b, :, :ctx + lens[b]], kv[1].v_cache[:, b, :, :ctx + lens[b]])
        assert np.isfinite(last[b]).all()
        assert nxt[b] == argmax_low(last[b]) or _margin(last[b]) < 2e-4, b     # (both sides within 1e-4 of exact logits)


def _handle_of_sizes(cfg):
    """A model handle that is asked for sizes only: every weight pointer is the same few bytes."""
    from paper_2401_12522_amd import binding as B
    some = torch.zeros(256, dtype=torch.uint8, device="cuda")
    w, handle = B._Weights(), B.C.c_void_p()
    for name, kind in B._Weights._fields_:
        setattr(w, name, some.data_ptr() if kind is B.C.c_void_p else (B.C.c_void_p * 1)(some.data_ptr()))
    c = B._Config(1, cfg.d_model, cfg.n_heads, cfg.n_kv_heads, cfg.head_dim, cfg.d_ffn, cfg.vocab, cfg.n_prompt, cfg.n_mask, 16,
                  cfg.rms_eps, cfg.rope_theta)
    B._check(B.lib().bita_model_create(B.C.byref(c), B.C.byref(w), B.C.byref(handle)))
    return handle


@pytest.mark.parametrize("cfg_name,over", [("tiny_gqa", {}), ("7b", {}), ("13b", {}), ("70b", {}), ("7b", dict(vocab=512))])
@pytest.mark.parametrize("batch", [1, 2, 3, 4])
def test_the_workspace_of_a_chunk_size_holds_every_shorter_chunk(bita, cfg_name, over, batch):
    """A pass of fewer rows may need more than one of more (more k splits): what a prefill of some chunk size is given has
    to hold any last chunk."""
    from paper_2401_12522_amd import binding as B
    handle, longest = _handle_of_sizes(synth.get_config(cfg_name, n_layers=1, **over)), 512 // batch
    try:
        needs = [B.lib().bita_workspace_bytes(handle, batch, r) for r in range(1, longest + 1)]
        fewer_need_more = [r for r in range(2, longest + 1) if needs[r - 1] < max(needs[:r - 1])]
        assert bool(fewer_need_more) == (cfg_name in ("7b", "13b") or (cfg_name, batch) == ("70b", 1))
        for chunk in fewer_need_more + [1, 17, longest]:
            for _ in range(2):
                assert B.lib().bita_prefill_workspace_bytes(handle, batch, chunk) >= max(needs[:chunk]) + needs[0], chunk
    finally:
        B.lib().bita_model_destroy(handle)


@pytest.mark.parametrize("cfg_name,chunk,n,batch", [("7b", 145, 289, 1), ("7b", 73, 145, 2), ("13b", 89, 177, 1)])
def test_a_last_chunk_that_needs_more_than_the_full_ones(bita, cfg_name, chunk, n, batch):
    """Widths where one row less than a chunk needs a larger workspace.  The call runs in the workspace it is given, as
    chunks of another size do, and one that is smaller than its own two chunk sizes need is refused before anything is enqueued."""
    from paper_2401_12522_amd import binding as B
    cfg = synth.get_config(cfg_name, n_layers=1)
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=4, device="cuda"), max_pos=512)
    assert model.workspace_bytes(batch, n % chunk) > model.workspace_bytes(batch, chunk)
    toks = dev_i32(np.random.default_rng(n).integers(0, cfg.vocab, size=(batch, n)))
    kv, other = bita.KVState(cfg, 1, batch, 512, chunk), bita.KVState(cfg, 1, batch, 512, 64)
    ws = bita.prefill_workspace(model, batch, chunk)
    bita.prefill(model, kv, 0, toks, chunk, workspace=ws)
    bita.prefill(model, other, 0, toks, 64)
    torch.cuda.synchronize()
    assert kv.ctx_len.tolist() == other.ctx_len.tolist() == [n] * batch
    for a, b in ((kv.k_cache, other.k_cache), (kv.v_cache, other.v_cache)):
        assert bool(((a.float() - b.float()).abs() <= 2.0 ** -7 * b.float().abs() + 1e-5).all())   # one unit of bf16
    kv.ctx_len.zero_()
    rc = B.lib().bita_prefill(model.handle, B.C.byref(kv.desc(0)), B._ptr(toks), n, None, B._ptr(kv.ctx_len), batch, chunk,
                              B._ptr(ws), model.workspace_bytes(batch, n % chunk), None, B._stream())
    torch.cuda.synchronize()
    assert rc == -3 and kv.ctx_len.tolist() == [0] * batch       # (the tokens and the last rows need room of their own)

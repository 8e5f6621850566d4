"""Paged KV cache through the C ABI: the same step over a shuffled page pool must reproduce,
bit for bit, what the contiguous layout gives (only addresses differ), and a paged prefill +
decode matches the oracle like the contiguous one does."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.model import argmax_low
from gpu_util import dev_i32

pytestmark = pytest.mark.gpu

KV_TOL = 3e-2
MARGIN = 6e-2


@pytest.fixture(scope="module")
def bita():
    import paper_2401_12522_amd as b
    b.lib()
    return b


def _random_cache(kv, lens, seed):
    """Seeded N(0,1) bf16 K/V in slots below each sequence's length (contiguous layout)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    for b, n in enumerate(lens):
        shape = (kv.k_cache.shape[0], kv.k_cache.shape[2], n, kv.k_cache.shape[4])
        kv.k_cache[:, b, :, :n] = torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16)
        kv.v_cache[:, b, :, :n] = torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16)
        kv.ctx_len[b] = n


@pytest.mark.parametrize("cfg_name,n_layers,page,lens", [
    ("tiny", None, 16, [40, 64, 57]),          # pages smaller than a key chunk: every chunk gathers per lane
    ("tiny_gqa", None, 32, [75, 33, 128]),
    ("tiny", None, 64, [200, 1, 90]),
    ("7b", 1, 64, [300]),                      # head_dim 128, one query head per K/V head
    ("70b", 1, 128, [517, 260]),               # head_dim 128, paired query heads
])
def test_paged_steps_are_bit_identical_to_contiguous(bita, cfg_name, n_layers, page, lens):
    cfg = synth.get_config(cfg_name) if n_layers is None else synth.get_config(cfg_name, n_layers=n_layers)
    L = cfg.n_layers
    B = len(lens)
    w = synth.SynthWeights(cfg, seed=2, device="cuda")
    tin = synth.attach_mask_groups(synth.random_tree(12, 4, 1), [0], cfg.n_mask)
    smax = (max(lens) + 64 + page - 1) // page * page
    model = bita.Model(cfg, w, max_pos=smax + 64)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, cfg.n_mask)
    flat = bita.KVState(cfg, L, B, smax, tmpl.rows)
    paged = bita.PagedKVState(cfg, L, B, smax, tmpl.rows, page, n_pages=B * (smax // page) + 5, seed=7)
    _random_cache(flat, lens, 3)
    for b, n in enumerate(lens):
        paged.load_contiguous(b, flat.k_cache[:, b], flat.v_cache[:, b], n)
    bufs = [bita.StepBuffers(model, tmpl, B, tmpl.kmax, want_logits=True) for _ in range(2)]
    rng = np.random.default_rng(11)
    root = dev_i32(rng.integers(0, cfg.vocab, B))
    grown = list(lens)
    for step in range(3):
        cand = dev_i32(rng.integers(0, cfg.vocab, (B, cfg.n_mask, tmpl.kmax)))
        hint = max(grown)
        if step > 0:
            # a draft whose first level is accepted: score the tree once, plant the root's greedy
            # token as its first child, then run the step proper
            bita.build_tree(tmpl, root, cand, None, None, B, bufs[0].token)
            bita.verify_step(model, flat, hint, tmpl, bufs[0], B)
            cand[:, 0, 0] = bufs[0].argmax[:, 0]
        for kv, buf in ((flat, bufs[0]), (paged, bufs[1])):
            bita.decode_step(model, kv, hint, tmpl, buf, B, root, cand)
        torch.cuda.synchronize()
        a, p = bufs
        assert torch.isfinite(a.logits).all()
        assert torch.equal(a.logits, p.logits), (step, (a.logits - p.logits).abs().max().item())
        for name in ("token", "argmax", "topk_ids", "topk_val", "path", "n_acc", "bonus", "emitted", "next_group", "next_shift"):
            assert torch.equal(getattr(a, name), getattr(p, name)), (step, name)
        assert torch.equal(flat.ctx_len, paged.ctx_len)
        grown = flat.ctx_len.cpu().tolist()
        for b in range(B):
            k, v = paged.contiguous(b)
            assert torch.equal(k[:, :, :grown[b]], flat.k_cache[:, b, :, :grown[b]]), (step, b)
            assert torch.equal(v[:, :, :grown[b]], flat.v_cache[:, b, :, :grown[b]]), (step, b)
        assert step == 0 or int(a.n_acc.min()) >= 2
        root = a.bonus.clone()
    # pages no sequence owns were never written
    owned = set(paged.block_table.cpu().numpy().ravel().tolist())
    spare = [i for i in range(paged.n_pages) if i not in owned]
    assert spare and not paged.k_cache[:, spare].any() and not paged.v_cache[:, spare].any()


@pytest.mark.parametrize("page", [16, 64])
@pytest.mark.parametrize("cfg_name,lens,heads_wg", [("7b", [1400, 333, 1000, 77], 1), ("70b", [900, 128, 511], 8)])
def test_paged_steps_of_more_workgroups_than_cus(bita, cfg_name, lens, heads_wg, page):
    """64-node trees over several sequences of ragged lengths: four waves per workgroup, one head or eight, from pages as
    from contiguous rows; and every sequence as by itself, where a workgroup has a CU to itself and eight waves."""
    cfg = synth.get_config(cfg_name, n_layers=1)
    B, hint, smax = len(lens), max(lens), 1536
    tin = synth.attach_mask_groups(synth.full_branching_tree([4, 3, 2, 1], 64), [0], cfg.n_mask)
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=2, device="cuda"), max_pos=smax + 64)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, cfg.n_mask)
    plan = lambda b, n, **k: bita.binding.attention_plan_info(b, tmpl.rows, cfg.n_heads, cfg.n_kv_heads, 128, n, cfg.n_prompt, **k)   # noqa: E731
    for p in (plan(B, hint), plan(B, hint, page_size=page)):
        assert (p["waves"], p["heads"], p["splits"]) == (4, heads_wg, 1) and p["workgroups"] > 256
    flat = bita.KVState(cfg, 1, B, smax, tmpl.rows)
    paged = bita.PagedKVState(cfg, 1, B, smax, tmpl.rows, page, n_pages=B * (smax // page) + 5, seed=7)
    _random_cache(flat, lens, 3)
    for b, n in enumerate(lens):
        paged.load_contiguous(b, flat.k_cache[:, b], flat.v_cache[:, b], n)
    start = flat.k_cache.clone(), flat.v_cache.clone()
    rng = np.random.default_rng(11)
    root, cand = dev_i32(rng.integers(0, cfg.vocab, B)), dev_i32(rng.integers(0, cfg.vocab, (B, cfg.n_mask, tmpl.kmax)))
    a, p = [bita.StepBuffers(model, tmpl, B, tmpl.kmax, want_logits=True) for _ in range(2)]
    for kv, buf in ((flat, a), (paged, p)):
        bita.decode_step(model, kv, hint, tmpl, buf, B, root, cand)
    torch.cuda.synchronize()
    assert torch.isfinite(a.logits).all()
    assert torch.equal(a.logits, p.logits), (a.logits - p.logits).abs().max().item()
    for name in ("token", "argmax", "topk_ids", "topk_val", "path", "n_acc", "bonus", "emitted", "next_group", "next_shift"):
        assert torch.equal(getattr(a, name), getattr(p, name)), name
    for b in range(B):
        k, v = paged.contiguous(b)
        n = int(paged.ctx_len[b])
        assert n == int(flat.ctx_len[b]) > lens[b]
        assert torch.equal(k[:, :, :n], flat.k_cache[:, b, :, :n]) and torch.equal(v[:, :, :n], flat.v_cache[:, b, :, :n])
    one, buf = bita.KVState(cfg, 1, 1, smax, tmpl.rows), bita.StepBuffers(model, tmpl, 1, tmpl.kmax, want_logits=True)
    for b, n in enumerate(lens):
        assert plan(1, n)["waves"] == 8
        one.k_cache.copy_(start[0][:, b:b + 1])
        one.v_cache.copy_(start[1][:, b:b + 1])
        one.ctx_len.fill_(n)
        bita.decode_step(model, one, n, tmpl, buf, 1, root[b:b + 1].clone(), cand[b:b + 1].clone())
        torch.cuda.synchronize()
        ref, got = buf.logits[0].double(), a.logits[b].double()
        # each side's two-plane sums are within 1.3e-5 of 64 bits (measured at these widths), and within three times that of each other
        assert float((got - ref).norm() / ref.norm()) < 4e-5, b


@pytest.mark.parametrize("hd,heads,page_lg", [(128, 1, 23), (128, 1, 24), (128, 2, 24), (128, 1, 25), (64, 2, 24), (64, 1, 25)])
def test_pages_whose_bytes_leave_32_bits(bita, hd, heads, page_lg):
    """One page larger than the sequence, of 2, 4 or 8 GiB per K/V head (4 GiB and its multiples are zero
    in 32 bits): the step still equals the contiguous one bit for bit, over a context of several
    chunks per wave."""
    cfg = synth.get_config("tiny", n_layers=1, d_model=128, n_heads=heads, n_kv_heads=1, head_dim=hd, d_ffn=256)
    n = 900
    tin = synth.attach_mask_groups(synth.random_tree(12, 4, 1), [0], cfg.n_mask)
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=4, device="cuda"), max_pos=n + 128)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, cfg.n_mask)
    flat = bita.KVState(cfg, 1, 1, n + 64, tmpl.rows)
    paged = bita.PagedKVState(cfg, 1, 1, n + 64, tmpl.rows, 1 << page_lg)
    _random_cache(flat, [n], 5)
    paged.load_contiguous(0, flat.k_cache[:, 0], flat.v_cache[:, 0], n)
    bufs = [bita.StepBuffers(model, tmpl, 1, tmpl.kmax, want_logits=True) for _ in range(2)]
    rng = np.random.default_rng(13)
    root, cand = dev_i32(rng.integers(0, cfg.vocab, 1)), dev_i32(rng.integers(0, cfg.vocab, (1, cfg.n_mask, tmpl.kmax)))
    for kv, buf in ((flat, bufs[0]), (paged, bufs[1])):
        bita.decode_step(model, kv, n, tmpl, buf, 1, root, cand)
    torch.cuda.synchronize()
    assert torch.isfinite(bufs[0].logits).all()
    assert torch.equal(bufs[0].logits, bufs[1].logits), (bufs[0].logits - bufs[1].logits).abs().max().item()
    grown = int(flat.ctx_len[0])
    assert grown == int(paged.ctx_len[0]) > n
    assert torch.equal(paged.k_cache[0, 0, :, :grown], flat.k_cache[0, 0, :, :grown])
    assert torch.equal(paged.v_cache[0, 0, :, :grown], flat.v_cache[0, 0, :, :grown])


def test_paged_prefill_and_decode_against_oracle(bita):
    """Prompt -> pages -> tokens: the pages hold the oracle's causal-pass K/V and the stream is
    the oracle's greedy stream where its margins are decisive."""
    cfg = synth.get_config("tiny_gqa")
    tin = synth.attach_mask_groups(synth.random_tree(8, 3, 0), [0], cfg.n_mask)
    w = synth.SynthWeights(cfg, seed=0)
    om = oracle.OracleModel(cfg, w)
    d = oracle.tree.derive_template(tin.parent, tin.is_mask, tin.n_mask)
    smax, page, steps = 256, 32, 8
    model = bita.Model(cfg, w, max_pos=smax + 64)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, tin.n_mask)
    kv = bita.PagedKVState(cfg, cfg.n_layers, 1, smax, max(tmpl.rows, 48), page, seed=3)
    ctx = synth.random_context(cfg.vocab, 64, 105)          # a seed whose first 33 greedy margins are decisive
    first = bita.prefill(model, kv, 0, dev_i32(ctx[None]), 48)
    torch.cuda.synchronize()
    assert int(kv.ctx_len[0]) == len(ctx)
    n = len(ctx)
    ck, cv = oracle.decode.prefill(om, np.concatenate([ctx, [0]]))   # K/V of all n tokens
    gk, gv = kv.contiguous(0)
    for l in range(cfg.n_layers):
        assert np.abs(gk[l, :, :n].permute(1, 0, 2).double().cpu().numpy() - ck[l]).max() <= KV_TOL
        assert np.abs(gv[l, :, :n].permute(1, 0, 2).double().cpu().numpy() - cv[l]).max() <= KV_TOL
    # greedy reference stream
    ck, cv = oracle.decode.prefill(om, ctx)
    ref, margins, last = [], [], int(ctx[-1])
    for _ in range(steps * (d.tree_depth + 1) + 2):
        lg, k, v = oracle.forward_rows(om, [last], [0], [-1], [ck[0].shape[0]], [[0]], ck, cv)
        ck, cv = oracle.compact_kv(ck, cv, k, v, [0])
        last = argmax_low(lg[0])
        ref.append(last)
        s = np.sort(lg[0])
        margins.append(s[-1] - s[-2])
    emitted = [int(first[0])]
    kv.resize_rows(cfg.n_layers, cfg, tmpl.rows)
    buf = bita.StepBuffers(model, tmpl, 1, d.kmax)
    buf.bonus.copy_(first)
    buf.next_shift[0] = cfg.n_mask
    for t in range(steps):
        bita.decode_step(model, kv, n + t * (d.tree_depth + 1), tmpl, buf, 1, buf.bonus, buf.topk_ids, buf.next_group, buf.next_shift)
        torch.cuda.synchronize()
        emitted.extend(buf.emitted[0, : int(buf.n_acc[0])].cpu().tolist())
    low = [i for i in range(len(emitted)) if margins[i] <= MARGIN]
    upto = low[0] if low else len(emitted)
    assert upto >= 6, "seed gives an early near-tie; pick another"
    assert emitted[:upto] == ref[:upto]


def test_paged_descriptor_is_validated(bita):
    cfg = synth.get_config("tiny")
    w = synth.SynthWeights(cfg, seed=1)
    model = bita.Model(cfg, w, max_pos=256)
    tin = synth.attach_mask_groups(synth.random_tree(4, 2, 0), [0], cfg.n_mask)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, cfg.n_mask)
    kv = bita.PagedKVState(cfg, cfg.n_layers, 1, 128, tmpl.rows, 32)
    buf = bita.StepBuffers(model, tmpl, 1, tmpl.kmax)
    cand = dev_i32(np.zeros((1, cfg.n_mask, tmpl.kmax)))
    kv.page_size = 24                                       # not a power of two
    with pytest.raises(bita.BitaError) as e:
        bita.decode_step(model, kv, 0, tmpl, buf, 1, dev_i32([1]), cand)
    assert e.value.code == -1
    kv.page_size, kv.max_pages = 32, 2                      # table shorter than smax
    with pytest.raises(bita.BitaError) as e:
        bita.decode_step(model, kv, 0, tmpl, buf, 1, dev_i32([1]), cand)
    assert e.value.code == -3
    torch.cuda.synchronize()

"""Tree attention (GPU) where neighbouring row tiles of a head run as one workgroup whose waves share every chunk: two and four
tiles, several sequences of unequal lengths and one, last workgroups with missing tiles and rows, chunks at every edge, against the
formula in 64 bits."""
import math

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,lens,heads,chain,share,waves", [
    (68, [300, 0, 33, 129], 32, False, 2, 4),                               # two tiles, five tiles a head
    (68, [95, 96, 97, 1, 31], 32, False, 2, 4), (41, [64, 65, 63, 32, 31, 33, 2, 0], 32, False, 2, 4), (97, [200, 17, 90], 32, False, 2, 4),
    (68, [40, 300, 0, 1, 31, 32, 33, 64], 32, False, 4, 4),                 # four tiles, no key groups
    (256, [100, 77], 32, True, 2, 4), (250, [7, 161], 32, True, 2, 4),      # causal rows, two tiles
    (512, [0], 32, True, 4, 8), (490, [300], 32, True, 4, 8), (481, [1], 32, True, 4, 8), (379, [45], 40, True, 4, 8)])   # four tiles on eight waves
def test_tiles_that_share_chunks(rows, lens, heads, chain, share, waves):
    import paper_2401_12522_amd as bita
    hd, B, P, longest = 128, len(lens), 0 if chain else 5, max(lens)
    if chain:
        parent, is_mask, n_tree = np.arange(rows, dtype=np.int32) - 1, np.zeros(rows, np.uint8), rows
    else:
        tin = synth.attach_mask_groups(synth.random_tree(rows - 4, 4, rows), [0], 4)
        parent, is_mask, n_tree = tin.parent, tin.is_mask, tin.n_tree
    R = len(parent)
    plan = bita.binding.attention_plan_info(B, R, heads, heads, hd, longest, P)
    assert plan["waves"] == 4 and plan["splits"] == 1 and plan["workgroups"] > 512, plan
    launch = bita.binding.attention_launch_info(B, R, heads, heads, hd, longest, P)
    assert (launch["share"], launch["waves"]) == (share, waves), launch
    tmpl = bita.TreeTemplate(parent, is_mask, n_tree, 4)
    g = torch.Generator(device="cuda").manual_seed(rows + B)
    b16 = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)   # noqa: E731
    q, kt, vt = b16(B, R, heads, hd), b16(B, heads, R, hd), b16(B, heads, R, hd)
    kt_lo, vt_lo = (b16(B, heads, R, hd).float() / 512).to(torch.bfloat16), (b16(B, heads, R, hd).float() / 512).to(torch.bfloat16)
    kc, vc = b16(B, heads, longest + 1, hd), b16(B, heads, longest + 1, hd)
    kc[:, :, -1] = float("nan")                                              # a slot past every context is never read into a result
    pk, pv = (b16(heads, P, hd), b16(heads, P, hd)) if P else (None, None)
    hi, lo = bita.tree_attention(tmpl, q, kc, vc, kt, vt, pk, pv, torch.tensor(lens, dtype=torch.int32, device="cuda"), longest,
                                 k_tree_lo=kt_lo, v_tree_lo=vt_lo, two_plane_out=True)
    out = (hi.double() + lo.double()).view(B, R, heads, hd)
    inside = np.zeros((R, R), bool)
    for i, p in enumerate(parent):
        if p >= 0:
            inside[i] = inside[p]
        inside[i, i] = True
    inside, masks = torch.tensor(inside, device="cuda"), torch.tensor(np.asarray(is_mask).astype(bool), device="cuda")
    for b, n in enumerate(lens):
        seen = torch.cat([masks[:, None].expand(R, P), torch.ones(R, n, dtype=torch.bool, device="cuda"), inside], 1)
        for h in (0, heads // 2 + 1, heads - 1):
            keys = [kc[b, h, :n].double(), kt[b, h].double() + kt_lo[b, h].double()]
            vals = [vc[b, h, :n].double(), vt[b, h].double() + vt_lo[b, h].double()]
            if P:
                keys.insert(0, pk[h].double())
                vals.insert(0, pv[h].double())
            p = torch.softmax(((q[b, :, h].double() @ torch.cat(keys).T) / math.sqrt(hd)).masked_fill(~seen, -math.inf), -1)
            err = float((out[b, :, h] - p @ torch.cat(vals)).abs().max())
            assert err < 1e-4, (b, n, h, err)                                # the kernel tests' two-plane regression bound


@pytest.mark.parametrize("rows,lens,page,share,waves", [
    (68, [300, 0, 33, 129], 16, 2, 4), (68, [40, 300, 0, 1, 31, 32, 33, 64], 16, 4, 4), (97, [200, 17, 90, 128, 64, 65, 127, 63], 64, 4, 4),
    (512, [0], 16, 4, 8), (490, [300], 64, 4, 8), (481, [45], 32, 4, 8)])
def test_tiles_that_share_chunks_of_a_paged_cache(rows, lens, page, share, waves):
    """A pass over shuffled pages gives the rows of a pass over the contiguous cache bit for bit (page sizes below, at and above
    a chunk's, empty and full last pages)."""
    import paper_2401_12522_amd as bita
    cfg, B, smax = synth.get_config("7b", n_layers=1, d_model=256, vocab=512, d_ffn=256), len(lens), 384
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=6, device="cuda"), max_pos=1024)
    parent = np.arange(rows, dtype=np.int32) - 1 if B == 1 else synth.random_tree(rows, 4, rows)
    tmpl = bita.TreeTemplate(parent, np.zeros(rows, np.uint8), rows, cfg.n_mask)
    for ps in (0, page):
        launch = bita.binding.attention_launch_info(B, rows, cfg.n_heads, cfg.n_kv_heads, cfg.head_dim, max(lens), cfg.n_prompt, ps)
        assert (launch["share"], launch["waves"]) == (share, waves), launch
    flat, paged = bita.KVState(cfg, 1, B, smax, rows), bita.PagedKVState(cfg, 1, B, smax, rows, page, n_pages=B * (smax // page) + 3, seed=5)
    g = torch.Generator(device="cuda").manual_seed(rows)
    for b, n in enumerate(lens):
        flat.k_cache[:, b, :, :n] = torch.randn((1, cfg.n_kv_heads, n, cfg.head_dim), device="cuda", generator=g).to(torch.bfloat16)
        flat.v_cache[:, b, :, :n] = torch.randn((1, cfg.n_kv_heads, n, cfg.head_dim), device="cuda", generator=g).to(torch.bfloat16)
        paged.load_contiguous(b, flat.k_cache[:, b], flat.v_cache[:, b], n)
        flat.ctx_len[b] = n
    paged.ctx_len.copy_(flat.ctx_len)
    got = []
    for kv in (flat, paged):
        buf = bita.StepBuffers(model, tmpl, B, 1, want_logits=True)
        buf.token.copy_(torch.randint(0, cfg.vocab, tuple(buf.token.shape), dtype=torch.int32, generator=torch.Generator().manual_seed(1)))
        bita.verify_step(model, kv, max(lens), tmpl, buf, B)
        got.append(buf)
    torch.cuda.synchronize()
    assert torch.isfinite(got[0].logits).all()
    assert torch.equal(got[0].logits, got[1].logits) and torch.equal(flat.k_tree, paged.k_tree)

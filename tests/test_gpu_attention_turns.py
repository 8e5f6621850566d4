"""Tree attention (GPU) of several sequences of unequal lengths with grouped heads and more workgroups than the CUs hold at
once: a sequence's output does not depend on its place in the batch or on the others' lengths."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _in_any_place(rows, lens, hd, ranked):
    import paper_2401_12522_amd as bita
    heads, kv_heads, B, smax, P = 64, 8, len(lens), max(lens) + 1, 5
    tin = synth.attach_mask_groups(synth.random_tree(rows, 4, rows), [0], 4)
    R = tin.rows
    plan = bita.binding.attention_plan_info(B, R, heads, kv_heads, hd, max(lens), P)
    assert plan["workgroups"] > 512 and plan["waves"] == 4 and plan["heads"] > 1, plan
    assert bita.binding.attention_launch_info(B, R, heads, kv_heads, hd, max(lens), P)["ranked"] is ranked
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, 4)
    g = torch.Generator(device="cuda").manual_seed(rows + hd)
    b16 = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)   # noqa: E731
    q, kt, vt = b16(B, R, heads, hd), b16(B, kv_heads, R, hd), b16(B, kv_heads, R, hd)
    kc, vc, pk, pv = b16(B, kv_heads, smax, hd), b16(B, kv_heads, smax, hd), b16(kv_heads, P, hd), b16(kv_heads, P, hd)
    lens = torch.tensor(lens, dtype=torch.int32, device="cuda")

    def planes(at, hint):
        take = lambda t: t[at].contiguous()                                           # noqa: E731
        hi, lo = bita.tree_attention(tmpl, take(q), take(kc), take(vc), take(kt), take(vt), pk, pv, take(lens), hint, two_plane_out=True)
        return hi, lo
    here = planes(torch.arange(B), int(lens.max()))
    for perm in (torch.arange(B).flip(0), torch.tensor(np.random.default_rng(B).permutation(B))):
        there = planes(perm, int(lens.max()))
        for a, b in zip(here, there):
            assert torch.equal(a[perm], b)
    for b in range(B):                                   # and is what the sequence alone gives (other waves, other order of sums)
        hi, lo = planes(torch.tensor([b]), int(lens.max()))
        err = (here[0][b].double() + here[1][b].double() - hi[0].double() - lo[0].double()).abs().max()
        assert float(err) < 1e-4, (b, float(err))        # the kernel tests' two-plane regression bound


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("rows,lens", [(130, [40, 300]), (130, [77, 77]), (90, [5, 0, 400]), (70, [64, 64, 63, 65]), (41, [31, 500, 0, 500, 32, 33, 1]),
                                       (33, [1, 2, 3, 4, 5, 6, 7, 300]), (33, [300] * 8), (33, [9, 200, 8, 200, 7, 100, 200, 0])])
def test_a_sequence_in_any_place_of_the_batch(rows, lens, hd):
    _in_any_place(rows, lens, hd, False)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("rows,lens", [(68, [700, 1900, 0, 1900]), (170, [33, 2100]), (33, [1, 2000, 3, 4, 2500, 6, 7, 300]), (41, [2200] * 8),
                                       (60, [2000, 1, 2001, 1999, 2000]), (90, [5, 0, 2048])])
def test_sequences_that_start_longest_first(rows, lens, hd):
    _in_any_place(rows, lens, hd, True)


@pytest.mark.parametrize("rows,lens", [(68, [700, 1900, 0, 1900]), (33, [1, 2000, 3, 4, 2500, 6, 7, 300])])
def test_longest_first_on_a_paged_cache(rows, lens):
    """Eight waves per workgroup: the rows of passes over shuffled pages of two sizes, bit for bit, and, but for the order of
    the sums, those of a pass over the contiguous cache (four waves)."""
    import paper_2401_12522_amd as bita
    cfg, B, smax = synth.get_config("70b", n_layers=1, d_model=256, vocab=512, d_ffn=256), len(lens), 2560
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=6, device="cuda"), max_pos=4096)
    tmpl = bita.TreeTemplate(synth.random_tree(rows, 4, rows), np.zeros(rows, np.uint8), rows, cfg.n_mask)
    flat = bita.KVState(cfg, 1, B, smax, rows)
    g = torch.Generator(device="cuda").manual_seed(rows)
    for b, n in enumerate(lens):
        flat.k_cache[:, b, :, :n] = torch.randn((1, cfg.n_kv_heads, n, cfg.head_dim), device="cuda", generator=g).to(torch.bfloat16)
        flat.v_cache[:, b, :, :n] = torch.randn((1, cfg.n_kv_heads, n, cfg.head_dim), device="cuda", generator=g).to(torch.bfloat16)
        flat.ctx_len[b] = n
    logits = {}
    for page in (0, 16, 64):
        launch = bita.binding.attention_launch_info(B, rows, cfg.n_heads, cfg.n_kv_heads, cfg.head_dim, max(lens), cfg.n_prompt, page)
        assert launch["ranked"] and launch["waves"] == (8 if page else 4), launch
        kv = bita.PagedKVState(cfg, 1, B, smax, rows, page, seed=5) if page else flat
        for b, n in enumerate(lens if page else []):
            kv.load_contiguous(b, flat.k_cache[:, b], flat.v_cache[:, b], n)
        buf = bita.StepBuffers(model, tmpl, B, 1, want_logits=True)
        buf.token.copy_(torch.randint(0, cfg.vocab, tuple(buf.token.shape), dtype=torch.int32, generator=torch.Generator().manual_seed(1)))
        bita.verify_step(model, kv, max(lens), tmpl, buf, B)
        logits[page] = buf.logits
    torch.cuda.synchronize()
    assert torch.isfinite(logits[16]).all() and torch.equal(logits[16], logits[64])
    assert float((logits[0] - logits[16]).abs().max()) < 1e-4

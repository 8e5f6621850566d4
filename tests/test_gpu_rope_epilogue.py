"""QKV products with one k split rotate and store their columns themselves (GPU): the same rows, bit for bit, as the forms that leave
it to a kernel of its own, at ragged rows, several sequences, grouped heads, both head dimensions and every kind of launch."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _same_rows(cfg, rows, batch, variants):
    import paper_2401_12522_amd as bita
    from paper_2401_12522_amd import binding as B
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=4, device="cuda", norm_std=0.3), max_pos=1024)
    parent = np.maximum(np.arange(rows, dtype=np.int32) - np.random.default_rng(rows).integers(1, 4, rows), -1).astype(np.int32)
    parent[1:] = np.maximum(parent[1:], 0)
    tmpl = bita.TreeTemplate(parent, np.zeros(rows, np.uint8), rows, cfg.n_mask)
    kv = bita.KVState(cfg, cfg.n_layers, batch, 256, rows)
    kv.k_cache.normal_()
    kv.v_cache.normal_()
    kv.ctx_len.copy_(torch.arange(batch, dtype=torch.int32) * 37 + 11)
    buf = bita.StepBuffers(model, tmpl, batch, 1, want_logits=True)
    buf.token.copy_(torch.randint(0, cfg.vocab, tuple(buf.token.shape), dtype=torch.int32))

    def results(variant):
        buf.workspace.fill_(0x7F)                      # stale NaNs wherever a kernel does not write
        kv.k_tree.fill_(float("nan"))
        kv.v_tree.fill_(float("nan"))
        B.lib().bita_tune_gemm(variant, 1)
        try:
            bita.verify_step(model, kv, 128, tmpl, buf, batch)
        finally:
            B.lib().bita_tune_gemm(-1, -1)
        torch.cuda.synchronize()
        return [t.clone() for t in (kv.k_tree, kv.v_tree, buf.logits)]
    apart = results(10)                                # 6 waves: sums through memory, rotated behind them
    for t in apart:
        assert torch.isfinite(t).all()
    for v in variants:
        for a, b in zip(apart, results(v)):
            assert torch.equal(a, b), v


@pytest.mark.parametrize("name,over,rows,batch,variants", [
    ("tiny", {}, 1, 1, (8, 9)), ("tiny", {}, 12, 1, (8, 9)), ("tiny_gqa", {}, 20, 2, (8, 9)), ("tiny", {}, 68, 1, (8, 9)), ("tiny_gqa", {}, 25, 3, (8, 9)),
    ("tiny", {}, 33, 3, (8, 9)), ("tiny_gqa", {}, 75, 4, (8, 9, -1)),
    ("7b", dict(n_layers=1, vocab=512, d_ffn=512), 200, 2, (9, -1)), ("7b", dict(n_layers=1, vocab=512, d_ffn=512), 489, 1, (-1,)),
    ("13b", dict(n_layers=1, vocab=512, d_ffn=512), 505, 1, (-1,)), ("70b", dict(n_layers=1, vocab=512, d_ffn=512), 500, 1, (-1,))])
def test_rotated_columns_are_the_same(name, over, rows, batch, variants):
    _same_rows(synth.get_config(name, **over), rows, batch, variants)


@pytest.mark.parametrize("heads,kv_heads,hd,rows,batch,mt_pass,tiles", [
    (64, 64, 128, 161, 1, 6, 12), (64, 64, 64, 401, 1, 7, 12), (64, 8, 128, 481, 1, 8, 12), (40, 40, 128, 385, 1, 9, 12), (64, 64, 128, 289, 1, 10, 12),
    (64, 64, 128, 107, 3, 11, 12), (48, 48, 128, 257, 1, 6, 16), (40, 40, 128, 433, 1, 7, 16), (40, 40, 128, 449, 1, 8, 16),
    (48, 48, 128, 193, 2, 9, 16), (48, 48, 128, 431, 1, 9, 16)])
def test_rotated_columns_of_tall_launches(heads, kv_heads, hd, rows, batch, mt_pass, tiles):
    """Every number of m-tiles that a tall launch takes, the last pass with few rows, 16 and 12 weight tiles per workgroup."""
    from paper_2401_12522_amd import binding as B
    cfg = synth.get_config("7b", n_layers=1, d_model=512, n_heads=heads, n_kv_heads=kv_heads, head_dim=hd, vocab=512, d_ffn=512)
    B.lib().bita_tune_gemm(-1, 1)
    try:
        plan = B.gemm_plan_info(batch * rows, cfg.q_dim + 2 * cfg.kv_dim, cfg.d_model)
    finally:
        B.lib().bita_tune_gemm(-1, -1)
    assert (plan["splits"], plan["mt_pass"], plan["tall_tiles"]) == (1, mt_pass, tiles), plan
    _same_rows(cfg, rows, batch, (-1,))

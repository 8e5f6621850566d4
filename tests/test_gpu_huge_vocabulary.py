"""A vocabulary whose rows of logits, eight of them, are more than 4 GiB (GPU): the LM head's output stores
count 32-bit offsets from the first row of an instruction and would wrap in the last columns."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def test_logits_of_rows_past_four_gib():
    import paper_2401_12522_amd as bita
    from gpu_util import dev_i32
    V = (1 << 27) + 1024
    cfg = synth.get_config("tiny", n_layers=1, d_model=32, n_heads=1, n_kv_heads=1, d_ffn=64, vocab=V)
    w = synth.SynthWeights(cfg, seed=6, device="cuda")
    base = torch.randn(1 << 20, 32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).to(torch.bfloat16)
    table = base.repeat(V // (1 << 20) + 1, 1)[:V].contiguous()      # a table quickly made; the last columns are its first again
    w._store[("tok_emb", None)] = w._store[("lm_head", None)] = table
    model = bita.Model(cfg, w, max_pos=128)
    tin = synth.attach_mask_groups(synth.random_tree(12, 4, 1), [0], cfg.n_mask)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, cfg.n_mask)
    kv = bita.KVState(cfg, 1, 1, 64, tmpl.rows)
    kv.k_cache.normal_()
    kv.v_cache.normal_()
    kv.ctx_len.fill_(40)
    buf = bita.StepBuffers(model, tmpl, 1, 2, want_logits=True)
    rng = np.random.default_rng(2)
    buf.token.copy_(dev_i32(rng.integers(0, V, size=(1, tmpl.rows))))
    buf.token[:, tin.n_tree:] = torch.arange(cfg.n_mask, dtype=torch.int32, device="cuda")
    buf.logits.fill_(float("nan"))
    bita.verify_step(model, kv, 40, tmpl, buf, 1)
    torch.cuda.synchronize()
    first = buf.logits[0, :, :1 << 20]
    assert torch.isfinite(first).all() and float(first.abs().max()) > 1.0
    # equal weight rows give equal logits, bit for bit, wherever their columns lie
    for at in range(1 << 20, V, 1 << 20):
        part = buf.logits[0, :, at:at + (1 << 20)]
        assert torch.equal(part, first[:, :part.shape[1]]), at
    del model, buf, table, first, part, w
    torch.cuda.empty_cache()

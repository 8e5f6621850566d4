"""Rotation and scatter of the QKV sums (GPU) where the heads do not fill its workgroups: one step of two
layers against the oracle at head counts that leave a workgroup partly idle, with and without k splits."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev_i32, load_cache, round_state
from oracle.decode import BitaState, bita_step
from oracle.tree import derive_template

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv_heads,hd,rows", [(1, 1, 64, 1), (5, 5, 64, 9), (6, 3, 64, 8), (1, 1, 128, 5), (3, 1, 128, 20), (8, 4, 128, 33), (9, 3, 128, 2)])
def test_step_with_heads_that_leave_a_workgroup_partly_idle(heads, kv_heads, hd, rows):
    import paper_2401_12522_amd as bita
    cfg = synth.get_config("tiny", n_heads=heads, n_kv_heads=kv_heads, head_dim=hd)
    w = synth.SynthWeights(cfg, seed=heads, norm_std=0.3, prefix_std=1.0)
    tin = synth.attach_mask_groups(synth.random_tree(rows, 4, rows), [0], cfg.n_mask)
    d = derive_template(tin.parent, tin.is_mask, cfg.n_mask)
    om = oracle.OracleModel(cfg, w)
    st = round_state(BitaState(om, synth.random_context(cfg.vocab, 37, 0)))
    model = bita.Model(cfg, w, max_pos=128)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, cfg.n_mask)
    kv = bita.KVState(cfg, cfg.n_layers, 1, 64, tmpl.rows)
    Lc, root = load_cache(kv, st.cache_k, st.cache_v), st.root_token
    cand = np.random.default_rng(rows).integers(0, cfg.vocab, size=(cfg.n_mask, d.kmax)).astype(np.int32)
    ref = bita_step(om, d, st, cand)
    buf = bita.StepBuffers(model, tmpl, 1, d.kmax, want_logits=True)
    bita.decode_step(model, kv, Lc, tmpl, buf, 1, dev_i32([root]), dev_i32(cand[None]))
    torch.cuda.synchronize()
    assert np.abs(buf.logits[0].cpu().numpy() - ref["logits"]).max() <= 1e-4      # the small shape's regression bound of the step tests

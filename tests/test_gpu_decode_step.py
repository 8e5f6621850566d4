"""A step as one call (GPU) against its four calls, bit for bit: every output, the cache and the lengths, over tree
shapes, batches, groups and shifts, pages, accepted lengths from none to the tree's depth, sequences that end at the
cache's last slot, and a step that the cache has no room for."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev_i32

pytestmark = pytest.mark.gpu
OUTPUTS = ("token", "argmax", "topk_ids", "topk_val", "logits", "path", "n_acc", "bonus", "emitted", "next_group", "next_shift")
# model, sequences, rows; bytes for a pass of so many rows, and for a prefill in chunks of as many
WORKSPACES = [("tiny", 1, 12, 636160, 762112), ("tiny_gqa", 3, 20, 3072256, 3289600), ("tiny", 2, 1, 171008, 343296)]


def _four(bita, model, kv, hint, tmpl, buf, B, root, cand, group, shift):
    from paper_2401_12522_amd import binding as L
    L.build_tree(tmpl, root, cand, group, shift, B, buf.token)
    L.verify_step(model, kv, hint, tmpl, buf, B)
    L.accept(tmpl, buf, B)
    L.compact_kv(model, kv, hint, buf, B)


def _same(a, b, names):
    for n in names:
        x, y = getattr(a, n), getattr(b, n)
        assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x, y.view(torch.int16) if y.dtype == torch.bfloat16 else y), n


@pytest.mark.parametrize("cfg_name,tree,per_node,lens,page", [
    ("tiny", "one", None, [64], 0), ("tiny", "chain", False, [64], 0), ("tiny_gqa", "random", False, [40, 0, 57], 16), ("tiny", "random", True, [33, 1], 0),
    ("tiny_gqa", "wide", False, [31, 64, 7, 50, 12], 32), ("tiny", "long", None, [20], 0)])
def test_one_call_equals_four(cfg_name, tree, per_node, lens, page):
    import paper_2401_12522_amd as bita
    cfg = synth.get_config(cfg_name)
    w = synth.SynthWeights(cfg, seed=3)
    parent = {"one": np.array([-1], np.int32), "chain": np.arange(-1, 4).astype(np.int32), "random": synth.random_tree(21, 4, 2),
              "wide": synth.star_tree(90), "long": np.arange(-1, 69).astype(np.int32)}[tree]
    if per_node is None:
        is_mask, n_tree = np.zeros(len(parent), np.uint8), len(parent)
    else:
        t = synth.attach_mask_groups(parent, range(len(parent)) if per_node else [0], cfg.n_mask)
        parent, is_mask, n_tree = t.parent, t.is_mask, t.n_tree
    B, kmax = len(lens), 8
    tmpl = bita.TreeTemplate(parent, is_mask, n_tree, cfg.n_mask)
    groups = max(tmpl.n_groups, 1)
    smax = max(lens) + 3 * (tmpl.depth + 1)
    smax = -(-smax // page) * page if page else smax
    model = bita.Model(cfg, w, max_pos=smax + 80)
    rng = np.random.default_rng(len(lens))

    def states():
        g = torch.Generator(device="cuda").manual_seed(7)
        kv = bita.PagedKVState(cfg, cfg.n_layers, B, smax, tmpl.rows, page) if page else bita.KVState(cfg, cfg.n_layers, B, smax, tmpl.rows)
        kv.k_cache.copy_(torch.randn(kv.k_cache.shape, generator=g, device="cuda"))
        kv.v_cache.copy_(torch.randn(kv.v_cache.shape, generator=g, device="cuda"))
        kv.ctx_len.copy_(dev_i32(lens))
        buf = bita.StepBuffers(model, tmpl, B, kmax, want_logits=True)
        buf.workspace.fill_(0x5A)
        return kv, buf

    (kv1, b1), (kv4, b4) = states(), states()
    root, cand = dev_i32(rng.integers(0, cfg.vocab, B)), rng.integers(0, cfg.vocab, (B, groups * cfg.n_mask, kmax)).astype(np.int32)
    seen = set()
    for step in range(3):
        group, shift = (dev_i32(rng.integers(0, groups, B)), dev_i32(rng.integers(0, 2, B))) if step == 1 else (None, None)
        hint = int(kv1.ctx_len.max())
        if step != 1:
            # drafts that will be accepted: level by level, what the rows so far predict
            for lvl in range(min(cfg.n_mask, tmpl.depth)):
                from paper_2401_12522_amd import binding as L
                L.build_tree(tmpl, root, dev_i32(cand), None, None, B, b4.token)
                L.verify_step(model, kv4, hint, tmpl, b4, B)
                L.accept(tmpl, b4, B)
                for b in range(B):
                    if int(b4.n_acc[b]) == lvl + 1 and (b + step) % 3:
                        cand[b, lvl, 0] = int(b4.bonus[b])
        c = dev_i32(cand)
        bita.decode_step(model, kv1, hint, tmpl, b1, B, root, c, group, shift)
        _four(bita, model, kv4, hint, tmpl, b4, B, root, c, group, shift)
        torch.cuda.synchronize()
        _same(b1, b4, OUTPUTS)
        _same(kv1, kv4, ("ctx_len", "k_cache", "v_cache", "k_tree", "v_tree"))
        seen |= set(b1.n_acc.tolist())
        root = b1.bonus.clone()
    if tree in ("chain", "long"):
        assert max(seen) >= 4, seen


def test_a_full_cache_refuses_the_commit_alone():
    import paper_2401_12522_amd as bita
    cfg = synth.get_config("tiny")
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=3), max_pos=200)
    t = synth.attach_mask_groups(synth.random_tree(8, 3, 0), [0], cfg.n_mask)
    tmpl = bita.TreeTemplate(t.parent, t.is_mask, t.n_tree, cfg.n_mask)
    need = tmpl.depth + 1
    for room, refused in ((need, False), (need - 1, True)):
        got = []
        for call in ("one", "four"):
            kv = bita.KVState(cfg, cfg.n_layers, 1, 30 + room, tmpl.rows)
            kv.ctx_len.fill_(30)
            buf = bita.StepBuffers(model, tmpl, 1, 4, want_logits=True)
            root, cand = dev_i32([5]), dev_i32(np.arange(cfg.n_mask * 4).reshape(1, cfg.n_mask, 4))
            step = (lambda: bita.decode_step(model, kv, 30, tmpl, buf, 1, root, cand)) if call == "one" else \
                   (lambda: _four(bita, model, kv, 30, tmpl, buf, 1, root, cand, None, None))
            if refused:
                with pytest.raises(bita.BitaError, match="cache capacity"):
                    step()
            else:
                step()
            torch.cuda.synchronize()
            got.append((buf, kv))
        _same(got[0][0], got[1][0], OUTPUTS)
        _same(got[0][1], got[1][1], ("ctx_len", "k_cache", "v_cache"))
        assert int(got[0][1].ctx_len[0]) == 30 + (0 if refused else int(got[0][0].n_acc[0]))


@pytest.mark.parametrize("fault", ["workspace", "kmax", "position", "scratch rows"])
def test_what_the_pass_refuses_leaves_the_tokens_built(fault):
    """The pass refuses where the commit would not: the tokens are there all the same, nothing else is touched, and the
    message is the pass' own."""
    import paper_2401_12522_amd as bita
    cfg = synth.get_config("tiny_gqa")
    t = synth.attach_mask_groups(synth.random_tree(8, 3, 0), [0], cfg.n_mask)
    tmpl = bita.TreeTemplate(t.parent, t.is_mask, t.n_tree, cfg.n_mask)
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=3), max_pos=34 if fault == "position" else 200)
    rng = np.random.default_rng(1)
    root, cand = dev_i32(rng.integers(0, cfg.vocab, 2)), dev_i32(rng.integers(0, cfg.vocab, (2, cfg.n_mask, 4)))
    got = []
    for step in (lambda *a: bita.decode_step(*a, root, cand), lambda *a: _four(bita, *a, root, cand, None, None)):
        kv = bita.KVState(cfg, cfg.n_layers, 2, 64, tmpl.rows + (fault == "scratch rows"))
        kv.ctx_len.fill_(30)
        buf = bita.StepBuffers(model, tmpl, 2, 4, want_logits=True)
        for n in OUTPUTS:
            getattr(buf, n).fill_(-7)
        if fault == "workspace":
            buf.workspace = buf.workspace[:1024]
        if fault == "kmax":
            buf.kmax = 99
        with pytest.raises(bita.BitaError, match="bita_verify_step"):
            step(model, kv, 30, tmpl, buf, 2)
        torch.cuda.synchronize()
        got.append((buf, kv))
    _same(got[0][0], got[1][0], OUTPUTS)
    _same(got[0][1], got[1][1], ("ctx_len", "k_cache", "v_cache"))
    assert got[0][0].token[:, 0].tolist() == root.tolist() and int(got[0][0].n_acc[0]) == -7


@pytest.mark.parametrize("cfg_name,batch,rows,step_bytes,prefill_bytes", WORKSPACES)
def test_a_step_needs_the_pass_workspace_and_no_more(cfg_name, batch, rows, step_bytes, prefill_bytes):
    """Workspaces laid out for the pass alone hold the whole step: their sizes are what they were before there was a
    call for it, and nothing is written behind them."""
    import paper_2401_12522_amd as bita
    from paper_2401_12522_amd import binding as L
    cfg = synth.get_config(cfg_name)
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=3), max_pos=200)
    assert model.workspace_bytes(batch, rows) == step_bytes
    assert L.lib().bita_prefill_workspace_bytes(model.handle, batch, rows) == prefill_bytes
    parent = synth.random_tree(rows, 3, 0)
    tmpl = bita.TreeTemplate(parent, np.zeros(rows, np.uint8), rows, cfg.n_mask)
    rng = np.random.default_rng(rows)
    root, cand = dev_i32(rng.integers(0, cfg.vocab, batch)), dev_i32(rng.integers(0, cfg.vocab, (batch, cfg.n_mask, 4)))
    got = []
    for step in (lambda *a: bita.decode_step(*a, root, cand), lambda *a: _four(bita, *a, root, cand, None, None)):
        kv = bita.KVState(cfg, cfg.n_layers, batch, 100, rows)
        kv.ctx_len.copy_(dev_i32(np.arange(batch) * 9 + 5))
        buf = bita.StepBuffers(model, tmpl, batch, 4, want_logits=True)
        memory = torch.full((step_bytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        buf.workspace = memory[:step_bytes]
        step(model, kv, int(kv.ctx_len.max()), tmpl, buf, batch)
        torch.cuda.synchronize()
        assert bool((memory[step_bytes:] == 0x5A).all())
        got.append((buf, kv))
    _same(got[0][0], got[1][0], [n for n in OUTPUTS if not n.startswith("topk")])
    _same(got[0][1], got[1][1], ("ctx_len", "k_cache", "v_cache"))


def test_outputs_of_a_step_feed_the_next_in_a_graph():
    import paper_2401_12522_amd as bita
    cfg = synth.get_config("tiny_gqa")
    model = bita.Model(cfg, synth.SynthWeights(cfg, seed=5), max_pos=400)
    t = synth.attach_mask_groups(synth.random_tree(8, 3, 0), [0], cfg.n_mask)
    tmpl = bita.TreeTemplate(t.parent, t.is_mask, t.n_tree, cfg.n_mask)
    ends = []
    for graph in (False, True):
        kv = bita.KVState(cfg, cfg.n_layers, 2, 300, tmpl.rows)
        buf = bita.StepBuffers(model, tmpl, 2, 4, want_logits=True)
        step = lambda: bita.decode_step(model, kv, 200, tmpl, buf, 2, buf.bonus, buf.topk_ids, buf.next_group, buf.next_shift)   # noqa: E731
        step()
        torch.cuda.synchronize()
        buf.bonus.copy_(dev_i32([3, 9]))
        buf.next_group.zero_()
        buf.next_shift.copy_(dev_i32([4, 4]))
        kv.ctx_len.copy_(dev_i32([17, 40]))
        tokens = []
        if graph:
            gr = torch.cuda.CUDAGraph()
            with torch.cuda.graph(gr):
                step()
        for _ in range(6):
            gr.replay() if graph else step()
            torch.cuda.synchronize()
            tokens.append(buf.emitted.clone())
        ends.append((tokens, buf, kv))
    for a, b in zip(ends[0][0], ends[1][0]):
        assert torch.equal(a, b)
    _same(ends[0][1], ends[1][1], OUTPUTS)
    assert torch.equal(ends[0][2].ctx_len, ends[1][2].ctx_len)
    for b in range(2):
        n = int(ends[0][2].ctx_len[b])
        for x in ("k_cache", "v_cache"):
            assert torch.equal(getattr(ends[0][2], x)[:, b, :, 17:n], getattr(ends[1][2], x)[:, b, :, 17:n])

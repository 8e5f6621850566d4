"""What this framework's user has it do, as cases that can be timed and compared.

Five kinds of case, each through the package's public calls:

  decode     the four calls of a decode step (build the tree, verify pass, acceptance, commit),
             eagerly, on a model of the repository's shapes with one or two of its layers and its
             LM head: what a serving loop repeats for every emitted token
  prefill    the context brought into the cache by chunked causal passes
  gemm       one weight-streaming product alone, single-plane or two-plane activations
  attention  tree-masked attention alone (contiguous cache)
  select     greedy tokens and top-k candidates from given logits

Weights, caches and inputs are seeded random data of the shapes in synth/configs.py."""
import math
import random

import numpy as np
import torch

import paper_2401_12522_amd as bita
import synth
from paper_2401_12522_amd import binding


def listed():
    return [
        # The smallest whole step: two narrow layers, 8 draft rows and one mask group on a 64-token
        # context.  Nothing in it is large; launches and latency are all there is.
        dict(name="decode-tiny", kind="decode", model="tiny", layers=2, tree="random", tree_rows=8, per_node=False,
             batch=1, ctx_lo=64, ctx_hi=64, page=0, kmax=4),
        # The step the benchmark is quoted on: LLaMA-2-7B widths, 64-node tree and 4 mask rows, 1024-token context.
        dict(name="decode-7b", kind="decode", model="7b", layers=2, tree="full", tree_rows=64, per_node=False,
             batch=1, ctx_lo=1024, ctx_hi=1024, page=0, kmax=4),
        # The same step at 70B widths (grouped-query attention), 2048-token context.
        dict(name="decode-70b", kind="decode", model="70b", layers=1, tree="full", tree_rows=64, per_node=False,
             batch=1, ctx_lo=2048, ctx_hi=2048, page=0, kmax=4),
        # One token per pass: plain decoding, and what a drafting step falls back to.
        dict(name="decode-7b-one-row", kind="decode", model="7b", layers=2, tree="one", tree_rows=1, per_node=None,
             batch=1, ctx_lo=1024, ctx_hi=1024, page=0, kmax=1),
        # The paper's efficient tree (n*k+1 rows) with its mask group, odd row count, 13B widths, odd context.
        dict(name="decode-13b-efficient", kind="decode", model="13b", layers=1, tree="efficient", tree_rows=21,
             per_node=False, batch=1, ctx_lo=777, ctx_hi=777, page=0, kmax=5),
        # Several sequences per step, contexts of different lengths, paged cache (272 rows through every matrix).
        dict(name="decode-7b-batch4-paged", kind="decode", model="7b", layers=1, tree="full", tree_rows=64,
             per_node=False, batch=4, ctx_lo=700, ctx_hi=1400, page=64, kmax=4),
        # A mask group behind every draft node (170 rows), the paper's own placement.
        dict(name="decode-7b-pernode", kind="decode", model="7b", layers=1, tree="full", tree_rows=34, per_node=True,
             batch=1, ctx_lo=1024, ctx_hi=1024, page=0, kmax=3),
        # A prompt that does not divide into chunks: 512 + 488 rows.
        dict(name="prefill-7b", kind="prefill", model="7b", layers=2, batch=1, tokens_lo=1000, tokens_hi=1000, chunk=512),
        # The widest matrix of a 7B layer alone, activations as the step hands them over (two planes).
        dict(name="gemm-7b-gate-up", kind="gemm", m=68, n=22016, k=4096, planes=2),
        # A long-k product with one activation plane and an odd row count, no allocation in the call.
        dict(name="gemm-13b-down", kind="gemm", m=37, n=5120, k=13824, planes=1),
        # Attention by itself at the grouped-query shape: 8 sequences, contexts between 1024 and 4096 tokens.
        dict(name="attention-gqa-batch8", kind="attention", heads=64, kv_heads=8, head_dim=128, prompt=16,
             tree_rows=64, per_node=False, batch=8, ctx_lo=1024, ctx_hi=4096),
        # Selection by itself over the vocabulary of a step.
        dict(name="select-32000", kind="select", tree_rows=64, per_node=False, batch=1, vocab=32000, kmax=4),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "gemm", "gemm", "attention", "select"])
    if kind == "decode":
        model = rng.choice(["tiny", "tiny_gqa", "7b", "7b", "13b", "70b"])
        tree = rng.choice(["one", "random", "full", "efficient"])
        rows = {"one": 1, "random": _log_int(rng, 2, 100), "full": rng.randint(8, 64), "efficient": 4 * rng.randint(1, 8) + 1}[tree]
        per_node = None if tree == "one" else (rows <= 34 and rng.random() < 0.25)
        total = rows if per_node is None else rows + 4 * (rows if per_node else 1)
        batch = max(1, min(rng.choice([1, 1, 2, 3, 5]), (160 if model == "70b" else 280) // total))
        lo = _log_int(rng, 16, 2048)
        hi = lo if batch == 1 else min(3000, lo + rng.randint(0, lo))
        # the smallest step that can be measured keeps one token per row of k
        return dict(kind="decode", model=model, layers=rng.choice([1, 2]) if model in ("tiny", "tiny_gqa", "7b") else 1,
                    tree=tree, tree_rows=rows, per_node=per_node, batch=batch, ctx_lo=lo, ctx_hi=hi,
                    page=rng.choice([0, 0, 16, 64]), kmax=1 if tree == "one" else rng.randint(2, 8))
    if kind == "prefill":
        model = rng.choice(["tiny", "tiny_gqa", "7b", "13b"])
        batch = rng.choice([1, 1, 2])
        hi = _log_int(rng, 20, 800 // batch)
        return dict(kind="prefill", model=model, layers=1 if model == "13b" else 2, batch=batch,
                    tokens_lo=hi if batch == 1 else max(1, hi // 2), tokens_hi=hi,
                    chunk=min(rng.choice([64, 100, 256, 512]), 512 // batch))
    if kind == "gemm":
        n = 16 * _log_int(rng, 4, 3584)
        k = 8 * _log_int(rng, 16, max(17, min(3584, 230_000_000 // n // 8)))
        return dict(kind="gemm", m=_log_int(rng, 1, 512), n=n, k=k, planes=rng.choice([1, 2, 2]))
    if kind == "attention":
        heads, kv = rng.choice([(4, 4), (4, 2), (32, 32), (40, 40), (64, 8)])
        batch = rng.choice([1, 2, 4, 8])
        lo = _log_int(rng, 16, 4096 if batch <= 4 else 2048)
        return dict(kind="attention", heads=heads, kv_heads=kv, head_dim=64 if heads == 4 else 128,
                    prompt=rng.choice([0, 8, 16]), tree_rows=_log_int(rng, 1, 96), per_node=False, batch=batch,
                    ctx_lo=lo, ctx_hi=min(4096, lo + rng.randint(0, lo)))
    return dict(kind="select", tree_rows=_log_int(rng, 2, 64), per_node=False, batch=rng.choice([1, 2, 4]),
                vocab=16 * _log_int(rng, 16, 4000), kmax=rng.randint(1, 8))


# ------------------------------------------------------------------------------------------------ inputs
N_MASK = 4


def _tree_parents(case):
    t, rows = case.get("tree", "full"), case["tree_rows"]
    if t == "one":
        return np.array([-1], np.int32)
    if t == "efficient":
        return synth.efficient_tree_parents(4, (rows - 1) // 4)
    if t == "random":
        return synth.random_tree(rows, 6, rows)
    ks = [4, 3, 2, 1] if rows > 34 else [3, 2, 2, 1]
    full = synth.full_branching_tree(ks, rows)
    return full if len(full) == rows else synth.random_tree(rows, 6, rows)


def _layout(case):
    """(parent, is_mask, number of tree rows, mask tokens per group) of the pass."""
    tree = _tree_parents(case)
    if case["per_node"] is None:
        return tree, np.zeros(len(tree), np.uint8), len(tree), N_MASK
    t = synth.attach_mask_groups(tree, range(len(tree)) if case["per_node"] else [0], N_MASK)
    return t.parent, t.is_mask, t.n_tree, N_MASK


def _lengths(case, seed, lo, hi):
    r = random.Random(seed * 7 + 1)
    return [hi] + [r.randint(lo, hi) for _ in range(case["batch"] - 1)]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1009 + 17)
    return g


def _randn(g, *shape, scale=1.0):
    return (torch.randn(shape, generator=g, device="cuda") * scale).to(torch.bfloat16)


def _planes(g, *shape):
    """A random operand as the framework hands it on: bf16 value and bf16 rounding residual."""
    x = torch.randn(shape, generator=g, device="cuda")
    hi = x.to(torch.bfloat16)
    return hi, (x - hi.float()).to(torch.bfloat16)


def _weights(case, seed):
    cfg = synth.get_config(case["model"], n_layers=case["layers"])
    return cfg, synth.SynthWeights(cfg, seed=int(seed), device="cuda", norm_std=0.3)


def _caches(case, cfg, seed, lens):
    """The cached keys and values of every sequence, [layers][kv heads][length][head dim]."""
    g = _gen(seed)
    return [(_randn(g, cfg.n_layers, cfg.n_kv_heads, n, cfg.head_dim), _randn(g, cfg.n_layers, cfg.n_kv_heads, n, cfg.head_dim))
            for n in lens]


def _step_inputs(case, cfg, seed):
    r = np.random.default_rng(int(seed) + 5)
    root = r.integers(0, cfg.vocab, size=case["batch"]).astype(np.int32)
    groups = case["tree_rows"] if case["per_node"] else 1
    cand = r.integers(0, cfg.vocab, size=(case["batch"], groups * N_MASK, case["kmax"])).astype(np.int32)
    return root, cand


def prepare(case, seed):
    s = dict(kind=case["kind"])
    if case["kind"] in ("decode", "prefill"):
        cfg, w = _weights(case, seed)
        if case["kind"] == "decode":
            parent, is_mask, n_tree, n_mask = _layout(case)
            lens, rows = _lengths(case, seed, case["ctx_lo"], case["ctx_hi"]), len(parent)
            most = max(lens) + len(parent) + 16
            model = bita.Model(cfg, w, max_pos=most, free_source=True)
            tmpl = bita.TreeTemplate(parent, is_mask, n_tree, n_mask)
            smax = -(-most // 64) * 64
            kv = (bita.PagedKVState(cfg, cfg.n_layers, case["batch"], smax, rows, case["page"], seed=int(seed)) if case["page"]
                  else bita.KVState(cfg, cfg.n_layers, case["batch"], smax, rows))
            for b, (k, v) in enumerate(_caches(case, cfg, seed, lens)):
                if case["page"]:
                    kv.load_contiguous(b, k, v, lens[b])
                else:
                    kv.k_cache[:, b, :, :lens[b]] = k
                    kv.v_cache[:, b, :, :lens[b]] = v
            buf = bita.StepBuffers(model, tmpl, case["batch"], case["kmax"], want_logits=True)
            # the step's whole-number results side by side, so that a loop fetches them with one copy
            names = ("token", "argmax", "topk_ids", "path", "n_acc", "bonus", "emitted", "next_group", "next_shift")
            whole = torch.zeros(sum(getattr(buf, n).numel() for n in names), dtype=torch.int32, device="cuda")
            at = 0
            for n in names:
                t = getattr(buf, n)
                setattr(buf, n, whole[at:at + t.numel()].view(t.shape))
                at += t.numel()
            root, cand = _step_inputs(case, cfg, seed)
            s.update(model=model, tmpl=tmpl, kv=kv, buf=buf, whole=whole, batch=case["batch"], hint=max(lens),
                     lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), masks=tmpl.n_groups > 0,
                     root=torch.tensor(root, device="cuda"), cand=torch.tensor(cand, device="cuda"))
        else:
            lens = _lengths(case, seed, case["tokens_lo"], case["tokens_hi"])
            model = bita.Model(cfg, w, max_pos=max(lens) + 16, free_source=True)
            bita.prefill_prepare(model, max(lens), case["chunk"])
            kv = bita.KVState(cfg, cfg.n_layers, case["batch"], max(lens) + 16, case["chunk"])
            s.update(model=model, kv=kv, chunk=case["chunk"], tokens=torch.tensor(_prompt(case, cfg, seed), device="cuda"),
                     lens=torch.tensor(lens, dtype=torch.int32, device="cuda") if case["batch"] > 1 else None,
                     ws=bita.prefill_workspace(model, case["batch"], case["chunk"]),
                     next=torch.full((case["batch"],), -1, dtype=torch.int32, device="cuda"))
    elif case["kind"] == "gemm":
        a, a_lo, w = _gemm_inputs(case, seed)
        # the call that needs no workspace where its scratch holds the shape, as a loop that cannot allocate uses it
        fits = binding.lib().bita_gemm_noalloc_scratch_bytes(case["m"], case["n"], case["k"]) <= binding.lib().bita_gemm_noalloc_max_scratch_bytes()
        s.update(a=a, a_lo=a_lo, w=bita.pack_weight(w), n=case["n"],
                 out=torch.empty((case["m"], case["n"]), device="cuda") if case["planes"] == 1 and fits else None)
    elif case["kind"] == "attention":
        s.update(_attention_inputs(case, seed))
        parent, is_mask, n_tree, n_mask = _layout(case)
        s["tmpl"] = bita.TreeTemplate(parent, is_mask, n_tree, n_mask)
    else:
        parent, is_mask, n_tree, n_mask = _layout(case)
        s.update(tmpl=bita.TreeTemplate(parent, is_mask, n_tree, n_mask), kmax=case["kmax"], logits=_logits(case, seed))
    return s


def _prompt(case, cfg, seed):
    return np.random.default_rng(int(seed) + 9).integers(0, cfg.vocab, size=(case["batch"], case["tokens_hi"])).astype(np.int32)


def _gemm_inputs(case, seed):
    g = _gen(seed)
    a, a_lo = _planes(g, case["m"], case["k"])
    return a, (a_lo if case["planes"] == 2 else None), _randn(g, case["n"], case["k"], scale=0.02)


def _attention_inputs(case, seed):
    g, B, hd, P = _gen(seed), case["batch"], case["head_dim"], case["prompt"]
    R, kvh = len(_layout(case)[0]), case["kv_heads"]
    lens = _lengths(case, seed, case["ctx_lo"], case["ctx_hi"])
    q, q_lo = _planes(g, B, R, case["heads"], hd)
    kt, kt_lo = _planes(g, B, kvh, R, hd)
    vt, vt_lo = _planes(g, B, kvh, R, hd)
    smax = max(lens) + R
    return dict(q=q, q_lo=q_lo, k_tree=kt, k_tree_lo=kt_lo, v_tree=vt, v_tree_lo=vt_lo, k_cache=_randn(g, B, kvh, smax, hd),
                v_cache=_randn(g, B, kvh, smax, hd), prompt_k=_randn(g, kvh, P, hd) if P else None,
                prompt_v=_randn(g, kvh, P, hd) if P else None, hint=max(lens),
                lens=torch.tensor(lens, dtype=torch.int32, device="cuda"))


def _logits(case, seed):
    return torch.randn((case["batch"], len(_layout(case)[0]), case["vocab"]), generator=_gen(seed), device="cuda") * 1.5


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    if s["kind"] == "decode":
        # back to the same context (a loop would go on from the advanced one)
        s["kv"].ctx_len.copy_(s["lens"])
        bita.decode_step(s["model"], s["kv"], s["hint"], s["tmpl"], s["buf"], s["batch"], s["root"], s["cand"] if s["masks"] else None)
        return dict(logits=s["buf"].logits, k_rows=s["kv"].k_tree, v_rows=s["kv"].v_tree, whole=s["whole"], ctx_len=s["kv"].ctx_len)
    if s["kind"] == "prefill":
        s["kv"].ctx_len.zero_()
        token = bita.prefill(s["model"], s["kv"], 0, s["tokens"], s["chunk"], seq_len=s["lens"], workspace=s["ws"], next_token=s["next"])
        return dict(k_cache=s["kv"].k_cache, v_cache=s["kv"].v_cache, ctx_len=s["kv"].ctx_len, next_token=token)
    if s["kind"] == "gemm":
        if s["out"] is not None:
            return binding.gemm_noalloc(s["a"], s["w"], s["n"], s["out"], a_lo=s["a_lo"])
        return bita.gemm(s["a"], s["w"], s["n"], a_lo=s["a_lo"])
    if s["kind"] == "attention":
        return bita.tree_attention(s["tmpl"], s["q"], s["k_cache"], s["v_cache"], s["k_tree"], s["v_tree"], s["prompt_k"], s["prompt_v"],
                                   s["lens"], s["hint"], q_lo=s["q_lo"], k_tree_lo=s["k_tree_lo"], v_tree_lo=s["v_tree_lo"])
    return bita.select(s["tmpl"], s["logits"], s["kmax"])


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(bytes=2 * n * k + 2 * case["planes"] * m * k + 4 * m * n, flops=2 * m * n * k)
    tree_rows, per_node = case.get("tree_rows", 1), case.get("per_node", None)
    rows = tree_rows if per_node is None else tree_rows + N_MASK * (tree_rows if per_node else 1)
    B = case["batch"]
    if kind == "select":
        return dict(bytes=4 * B * rows * case["vocab"] + 4 * B * (tree_rows + 2 * N_MASK * case["kmax"]), flops=0)
    if kind == "attention":
        h, kvh, hd, P = case["heads"], case["kv_heads"], case["head_dim"], case["prompt"]
        ctx = (case["ctx_lo"] + case["ctx_hi"]) / 2 if B > 1 else case["ctx_hi"]
        return dict(bytes=2 * hd * (2 * B * kvh * ctx + 2 * kvh * P + 4 * B * kvh * rows + 3 * B * rows * h),
                    flops=4 * B * rows * h * hd * (ctx + rows / 2))
    cfg = synth.get_config(case["model"], n_layers=case["layers"])
    weights = cfg.weight_bytes()
    kv_row = 2 * 2 * cfg.kv_dim * cfg.n_layers
    if kind == "decode":
        ctx = (case["ctx_lo"] + case["ctx_hi"]) / 2 if B > 1 else case["ctx_hi"]
        return dict(bytes=weights + kv_row * (B * (ctx + rows) + cfg.n_prompt) + B * rows * (2 * cfg.d_model + 4 * cfg.vocab),
                    flops=B * rows * (weights + 4 * cfg.q_dim * cfg.n_layers * (ctx + rows / 2)))
    n = (case["tokens_lo"] + case["tokens_hi"]) / 2 if B > 1 else case["tokens_hi"]
    # every chunk passes over the weights of the layers; the last token alone needs the LM head
    chunks = -(-case["tokens_hi"] // case["chunk"])
    head = 2 * cfg.vocab * cfg.d_model
    return dict(bytes=weights + kv_row * B * n * (1 + (chunks - 1) / 2) + 2 * B * n * cfg.d_model,
                flops=B * n * (weights - head + 2 * cfg.q_dim * cfg.n_layers * n) + B * head)


def tolerance(case):
    """About four times what the same path gives with its sums taken in another order (other k splits and
    workgroup shapes; attention: against 64 bits rounded to bf16).  Rows and outputs kept as bf16 now and then
    round the other way, one unit of 2^-8 of the value or two; logits by themselves move by 1e-5."""
    if case["kind"] == "select":
        return "exact"
    if case["kind"] == "gemm":
        return {"rel": 2e-6, "max": 2e-5}           # seen: 4.1e-7 and 4.1e-6 (k = 4096), 3.7e-7 (k = 13824)
    if case["kind"] == "attention":
        return {"rel": 4e-4, "max": 1.6e-2}         # seen: 8.7e-5 and one unit
    if case["kind"] == "prefill":
        return {"rel": 1.2e-3, "max": 2e-2, "differ": 0.01}   # seen: 2.8e-4 and one unit
    return {"rel": 7e-4, "max": 2e-2, "differ": 0.01}         # seen: 1.7e-4, one unit, no whole value but a near-tie's rank


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def _rope(x, pos, theta):
    """x [rows][heads][hd] rotated by its row's position, pairs (i, i + hd/2)."""
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * theta ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / x.shape[-1])
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _norm(x, gain, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain.double()


def _attend(q, keys, values, seen, present):
    """q [rows][heads][hd], keys and values [kv heads][n][hd], seen [rows][n]; rows that are not present give zeros."""
    heads, hd = q.shape[1], q.shape[2]
    out = torch.zeros_like(q)
    for h in range(heads):
        g = h * keys.shape[0] // heads
        sc = (q[:, h] @ keys[g].T) / math.sqrt(hd)
        p = torch.softmax(sc.masked_fill(~seen, -math.inf), -1)
        out[:, h] = p @ values[g]
    return out * present[:, None, None]


def _forward(cfg, w, x, present, pos, is_mask, inside, cache):
    """Logits and the rows' keys and values of one sequence; cache[l] = (keys, values) [kv heads][n][hd], inside [rows][rows]."""
    R, hd = x.shape[0], cfg.head_dim
    new = []
    for l in range(cfg.n_layers):
        W = lambda n: w.torch(n, l).double()      # noqa: E731
        h = _norm(x, w.torch("attn_norm", l), cfg.rms_eps)
        q = _rope((h @ W("wq").T).view(R, cfg.n_heads, hd), pos, cfg.rope_theta)
        k = _rope((h @ W("wk").T).view(R, cfg.n_kv_heads, hd), pos, cfg.rope_theta).transpose(0, 1)
        v = (h @ W("wv").T).view(R, cfg.n_kv_heads, hd).transpose(0, 1)
        ck, cv = cache[l]
        pk, pv = w.torch("prompt_k", l).double(), w.torch("prompt_v", l).double()
        seen = torch.cat([is_mask[:, None].expand(R, pk.shape[1]), torch.ones(R, ck.shape[1], dtype=torch.bool, device=x.device), inside], 1)
        a = _attend(q, torch.cat([pk, ck, k], 1), torch.cat([pv, cv, v], 1), seen, present)
        x = x + a.reshape(R, -1) @ W("wo").T
        h = _norm(x, w.torch("ffn_norm", l), cfg.rms_eps)
        x = x + (torch.nn.functional.silu(h @ W("w_gate").T) * (h @ W("w_up").T)) @ W("w_down").T
        new.append((k, v))
    return _norm(x, w.torch("final_norm"), cfg.rms_eps), new


def _ancestors(parent):
    inside = np.zeros((len(parent), len(parent)), bool)
    depth = np.zeros(len(parent), np.int64)
    for i, p in enumerate(parent):
        if p >= 0:
            inside[i], depth[i] = inside[p], depth[p] + 1
        inside[i, i] = True
    return inside, depth


def exact(case, seed):
    dev = torch.device("cuda")
    if case["kind"] == "gemm":
        a, a_lo, w = _gemm_inputs(case, seed)
        x = a.double() + (a_lo.double() if a_lo is not None else 0.0)
        return x @ w.double().T
    if case["kind"] == "select":
        parent, is_mask, n_tree, _ = _layout(case)
        order = torch.sort(_logits(case, seed)[:, n_tree:].double(), dim=-1, descending=True)[0]
        return (None, None, order[..., :case["kmax"]].contiguous())
    parent, is_mask, n_tree, n_mask = _layout(case) if case["kind"] != "prefill" else (None, None, None, None)
    if case["kind"] == "attention":
        s = _attention_inputs(case, seed)
        inside, _ = _ancestors(parent)
        inside, masks = torch.tensor(inside, device=dev), torch.tensor(is_mask.astype(bool), device=dev)
        out = []
        for b, n in enumerate(s["lens"].tolist()):
            R, P = len(parent), case["prompt"]
            keys = [s["k_cache"][b, :, :n].double(), s["k_tree"][b].double() + s["k_tree_lo"][b].double()]
            vals = [s["v_cache"][b, :, :n].double(), s["v_tree"][b].double() + s["v_tree_lo"][b].double()]
            if P:
                keys.insert(0, s["prompt_k"].double())
                vals.insert(0, s["prompt_v"].double())
            seen = torch.cat([masks[:, None].expand(R, P), torch.ones(R, n, dtype=torch.bool, device=dev), inside], 1)
            o = _attend(s["q"][b].double() + s["q_lo"][b].double(), torch.cat(keys, 1), torch.cat(vals, 1), seen,
                        torch.ones(R, device=dev, dtype=torch.float64))
            out.append(o.reshape(R, -1))
        return torch.stack(out)
    cfg, w = _weights(case, seed)
    emb, head = w.torch("tok_emb"), w.torch("lm_head")
    if case["kind"] == "decode":
        lens = _lengths(case, seed, case["ctx_lo"], case["ctx_hi"])
        root, cand = _step_inputs(case, cfg, seed)
        inside, depth = _ancestors(parent)
        is_mask = is_mask.astype(bool)
        masks_first, children = {}, {}
        logits, k_rows, v_rows = [], [], []
        index = np.zeros(len(parent), np.int64)      # a mask row's place in its group, a draft row's rank among its siblings
        for i, p in enumerate(parent):
            if i and is_mask[i]:
                index[i] = index[p] + 1 if is_mask[p] else 0
            elif i:
                index[i] = children.setdefault(int(p), 0)
                children[int(p)] += 1
        for b, (ck, cv) in enumerate(_caches(case, cfg, seed, lens)):
            x = torch.zeros(len(parent), cfg.d_model, dtype=torch.float64, device=dev)
            present = np.ones(len(parent), bool)
            for i in range(len(parent)):
                if is_mask[i]:
                    x[i] = w.torch("mask_emb")[index[i]].double()
                elif i == 0:
                    x[i] = emb[int(root[b])].double()
                elif depth[i] <= N_MASK and index[i] < case["kmax"]:
                    x[i] = emb[int(cand[b, depth[i] - 1, index[i]])].double()
                else:
                    present[i] = False
            h, new = _forward(cfg, w, x, torch.tensor(present, device=dev), torch.tensor(depth + lens[b], device=dev),
                              torch.tensor(is_mask, device=dev), torch.tensor(inside, device=dev),
                              [(ck[l].double(), cv[l].double()) for l in range(cfg.n_layers)])
            logits.append(h @ head.double().T)
            k_rows.append(torch.stack([k for k, _ in new]))
            v_rows.append(torch.stack([v for _, v in new]))
        return dict(logits=torch.stack(logits), k_rows=torch.stack(k_rows, 1), v_rows=torch.stack(v_rows, 1), whole=None, ctx_len=None)
    lens, tokens = _lengths(case, seed, case["tokens_lo"], case["tokens_hi"]), _prompt(case, cfg, seed)
    smax = max(lens) + 16
    k_all = torch.zeros(cfg.n_layers, case["batch"], cfg.n_kv_heads, smax, cfg.head_dim, dtype=torch.float64, device=dev)
    v_all = torch.zeros_like(k_all)
    for b, n in enumerate(lens):
        for at in range(0, n, case["chunk"]):
            m = min(case["chunk"], n - at)
            x = emb[torch.tensor(tokens[b, at:at + m].astype(np.int64), device=dev)].double()
            # a later chunk reads what the earlier ones left in the cache: 16-bit values
            cache = [(k_all[l, b, :, :at].to(torch.bfloat16).double(), v_all[l, b, :, :at].to(torch.bfloat16).double()) for l in range(cfg.n_layers)]
            _, new = _forward(cfg, w, x, torch.ones(m, dtype=torch.bool, device=dev), torch.arange(at, at + m, device=dev),
                              torch.zeros(m, dtype=torch.bool, device=dev), torch.ones(m, m, dtype=torch.bool, device=dev).tril(), cache)
            for l, (k, v) in enumerate(new):
                k_all[l, b, :, at:at + m], v_all[l, b, :, at:at + m] = k, v
    return dict(k_cache=k_all, v_cache=v_all, ctx_len=None, next_token=None)

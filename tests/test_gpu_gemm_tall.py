"""Tall row passes with 12 and with 16 weight tiles per workgroup (GPU): the launch heuristic takes the form
that a case names (0: passes of 5 m-tiles), alone and inside a step, at shapes with a ragged last m-tile, a last pass shorter than
the others, a ragged last column group, one and several k splits, and gated outputs that end inside a
k-step of the next product."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.model import silu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,tiles,mt_pass,splits", [
    (170, 22016, 512, 12, 6, 1), (272, 22016, 256, 12, 9, 1), (265, 22000, 288, 12, 9, 1), (488, 12288, 256, 12, 8, 1),
    (300, 12288, 256, 0, 0, 1), (300, 32000, 256, 12, 7, 1), (250, 22016, 96, 12, 8, 1), (105, 22016, 4096, 12, 7, 2), (265, 12288, 4096, 12, 9, 2),
    (81, 57344, 256, 16, 6, 1), (165, 27648, 256, 16, 6, 1), (257, 27648, 256, 16, 9, 1), (162, 15360, 2048, 16, 6, 2),
    (257, 10240, 4096, 16, 9, 3), (152, 40960, 256, 12, 10, 1), (145, 22016, 4096, 12, 10, 2), (309, 22016, 288, 12, 10, 1), (341, 22016, 96, 12, 11, 1),
    (176, 40960, 160, 12, 11, 1), (145, 19440, 4552, 12, 10, 2)])
def test_gemm_rows_of_twelve_tiles(M, N, K, tiles, mt_pass, splits):
    import paper_2401_12522_amd as bita
    plan = bita.binding.gemm_plan_info(M, N, K)
    assert (plan["tall_tiles"], plan["mt_pass"], plan["splits"]) == (tiles, mt_pass, splits), plan
    g = torch.Generator().manual_seed(N + K + M)
    a32 = torch.randn(M, K, generator=g)
    hi = a32.to(torch.bfloat16)
    lo = (a32 - hi.float()).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16)
    out = bita.gemm(hi.cuda(), bita.pack_weight(w.cuda()), N, a_lo=lo.cuda()).cpu().double()
    ref = (hi.double() + lo.double()) @ w.double().T
    scale = float(ref.abs().max())
    assert torch.isfinite(out).all()
    assert float((out - ref).abs().max()) <= 2e-5 * scale + 1e-6         # fp32 accumulation, as everywhere


@pytest.mark.parametrize("M,N,K,tiles,mt_pass,splits", [
    # both k groups at once: few k-steps a split, or one pass of 6
    (188, 4720, 11528, 12, 6, 5), (81, 22016, 4096, 12, 6, 2), (161, 4096, 11000, 16, 6, 8), (107, 12288, 4096, 16, 7, 5), (330, 4720, 3336, 16, 7, 4),
    (113, 12288, 4088, 16, 8, 5), (113, 15360, 5120, 16, 8, 4), (256, 4096, 11008, 16, 8, 8), (140, 12288, 4096, 12, 9, 4), (257, 10240, 4096, 16, 9, 3),
    # in turns
    (161, 10240, 8184, 16, 6, 3), (105, 22016, 4088, 12, 7, 2), (120, 22016, 4096, 12, 8, 2), (265, 12288, 4096, 12, 9, 2), (340, 8192, 28672, 16, 6, 2)])
def test_split_tall_launches_in_turns_and_both_at_once(M, N, K, tiles, mt_pass, splits):
    import paper_2401_12522_amd as bita
    plan = bita.binding.gemm_plan_info(M, N, K)
    assert (plan["tall_tiles"], plan["mt_pass"], plan["splits"]) == (tiles, mt_pass, splits), plan
    g = torch.Generator(device="cuda").manual_seed(N + K)
    a32, w = torch.randn(M, K, generator=g, device="cuda"), (torch.randn(N, K, generator=g, device="cuda") * 0.05).to(torch.bfloat16)
    hi = a32.to(torch.bfloat16)
    lo = (a32 - hi.float()).to(torch.bfloat16)
    out, ref = bita.gemm(hi, bita.pack_weight(w), N, a_lo=lo).double(), (hi.double() + lo.double()) @ w.double().T
    assert torch.isfinite(out).all()
    assert float((out - ref).abs().max()) <= 2e-5 * float(ref.abs().max()) + 1e-6         # fp32 accumulation, as everywhere


@pytest.mark.parametrize("M,N,K,variant,splits", [
    (300, 12288, 1280, 9, 1), (300, 12288, 1288, 9, 1), (300, 12288, 1320, 9, 1), (300, 12288, 1376, 9, 1), (300, 12288, 1400, 9, 1), (300, 12288, 1440, 9, 1),
    (222, 35072, 1280, 11, 1), (222, 35072, 1304, 11, 1), (236, 9600, 4096, 9, 2), (236, 9600, 4136, 9, 2), (488, 4096, 4104, 9, 2),   # (the last writes its sums through)
    (300, 12288, 1248, 9, 1), (300, 4096, 4096, 9, 4), (128, 4096, 11008, 9, 8), (302, 272, 20512, 9, 8)])     # too few k-steps, too few workgroups: both at once
def test_passes_of_five_in_turns_and_both_at_once(M, N, K, variant, splits):
    import paper_2401_12522_amd as bita
    plan = bita.binding.gemm_plan_info(M, N, K)
    assert (plan["variant"], plan["mt_pass"], plan["splits"]) == (variant, 0, splits), plan
    g = torch.Generator().manual_seed(N + K)
    a32 = torch.randn(M, K, generator=g)
    hi = a32.to(torch.bfloat16)
    lo = (a32 - hi.float()).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16)
    out = bita.gemm(hi.cuda(), bita.pack_weight(w.cuda()), N, a_lo=lo.cuda())
    ref = (hi.cuda().float().double() + lo.cuda().double()) @ w.cuda().double().T
    assert torch.isfinite(out).all()
    assert float((out.double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max()) + 1e-6         # fp32 accumulation, as everywhere


@pytest.mark.parametrize("M,N,planes", [(272, 22016, 2), (112, 57344, 2), (150, 4096, 2), (300, 12288, 2), (20, 22016, 1), (300, 12288, 1)])
@pytest.mark.parametrize("K", [32, 64, 96, 160, 224, 232])
def test_k_groups_in_turns_at_short_k(M, N, planes, K):
    """Fewer k-steps than pipeline stages, remainders of the pipeline's round, and a second k group with fewer k-steps
    than the first, or none: tall passes, passes of 5, one plane."""
    import paper_2401_12522_amd as bita
    g = torch.Generator().manual_seed(N + K + M)
    a32 = torch.randn(M, K, generator=g)
    hi = a32.to(torch.bfloat16)
    lo = (a32 - hi.float()).to(torch.bfloat16) if planes == 2 else None
    w = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16)
    out = bita.gemm(hi.cuda(), bita.pack_weight(w.cuda()), N, a_lo=lo.cuda() if planes == 2 else None).cpu().double()
    ref = (hi.double() + (lo.double() if planes == 2 else 0.0)) @ w.double().T
    assert torch.isfinite(out).all()
    assert float((out - ref).abs().max()) <= 2e-5 * float(ref.abs().max()) + 1e-6


@pytest.mark.parametrize("d_ffn,batch,tiles", [(11008, 4, 12), (10976, 3, 12), (11024, 4, 12), (6160, 8, 16), (6128, 8, 12), (11520, 5, 12), (11008, 5, 12)])
def test_gated_output_of_twelve_tile_workgroups(d_ffn, batch, tiles):
    """One layer with a wide FFN on passes of 68 rows x batch; the pass with the widths' own launch shapes
    against the same pass in the older forms (passes of 5 m-tiles), whose parity the step tests hold."""
    import paper_2401_12522_amd as bita
    from paper_2401_12522_amd import binding as B
    cfg = synth.get_config("tiny", d_ffn=d_ffn, n_layers=1)
    w = synth.SynthWeights(cfg, seed=2, device="cuda", norm_std=0.3)
    model = bita.Model(cfg, w, max_pos=256)
    tin = synth.attach_mask_groups(synth.full_branching_tree([4, 3, 2, 1], 64), [0], cfg.n_mask)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, cfg.n_mask)
    plan = B.gemm_plan_info(batch * tmpl.rows, 2 * d_ffn, cfg.d_model)
    assert (plan["tall_tiles"], plan["splits"]) == (tiles, 1), plan     # complete sums: the workgroup gates its own output
    kv = bita.KVState(cfg, 1, batch, 128, tmpl.rows)
    kv.k_cache.normal_()
    kv.v_cache.normal_()
    kv.ctx_len.fill_(50)
    buf = bita.StepBuffers(model, tmpl, batch, 4, want_logits=True)
    rng = np.random.default_rng(d_ffn)
    buf.token.copy_(torch.tensor(rng.integers(0, cfg.vocab, size=tuple(buf.token.shape)), dtype=torch.int32))
    buf.token[:, tin.n_tree:] = torch.arange(4, dtype=torch.int32, device="cuda")

    def logits():
        buf.workspace.fill_(0x7F)                       # stale NaNs wherever a kernel does not write
        bita.verify_step(model, kv, 50, tmpl, buf, batch)
        torch.cuda.synchronize()
        return buf.logits.double().cpu()
    got = logits()
    B.lib().bita_tune_gemm(-2, -1)
    try:
        ref = logits()
    finally:
        B.lib().bita_tune_gemm(-1, -1)
    assert torch.isfinite(got).all()
    assert float((got - ref).abs().max()) <= 1e-4       # the small shape's regression bound of the step tests
